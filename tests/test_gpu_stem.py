"""First layers of a network (few input channels, pixels staged in LDS): every channel count and tile shape they take, images of one pixel, rows as
wide as the staging allows and one wider (the generic kernels), against the oracle; and small tiles of the generic kernels."""
import numpy as np
import pytest

import workloads as wk
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu
H = parity.H

# input channels, output channels, images, height, width
STEMS = {"one_pixel": (3, 16, 2, 1, 1), "ragged": (3, 16, 2, 5, 7), "one_tile": (3, 16, 4, 8, 8), "one_channel": (1, 16, 2, 6, 9), "c32": (2, 32, 2, 9, 4),
         "c64_four_channels": (4, 64, 2, 7, 11), "c32_tiles": (3, 32, 9, 30, 31), "c64_tiles": (3, 64, 5, 31, 30), "widest": (3, 16, 3, 5, 127),
         "wider": (3, 16, 3, 5, 128), "many_trips": (3, 16, 130, 32, 32), "tall_many_channels": (5, 16, 2, 9, 8)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(STEMS))
def test_first_layer(H, which, dtype):
    import torch
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    cin, cout, N, h, w = STEMS[which]
    print(f"case first layer {which} {dtype}", flush=True)
    blocks = [(wk.BLOCK_STEM, cin, 0, cout, 1, 0)]
    mod = ddg.Module(make_desc(2, 1, N, (cin, h, w), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(2, [blocks], N, (cin, h, w), 0, 0.9, 0.0, 1e-5, "f64", k_first=1, store_bf16=(dtype == "bf16"))
    theta = (wk.normal(11, 1, mod.param_count()) * 0.2 + 0.05).astype(np.float32)
    mod.set_params(theta)
    oracle.set_params(1, theta.astype(np.float64))

    class WL:
        pass
    wl = WL(); wl.dtype = dtype
    for t in range(3):          # (from t = 1 on two minibatches a launch)
        x = wk.normal(13, t, N * cin * h * w).reshape(N, cin, h, w)
        d = wk.normal(17, t, N * cout * h * w).reshape(N, cout, h, w)
        xd, dd = H.to_dev_nhwc(x, wl), H.to_dev_nhwc(d, wl)
        x, d = H.from_dev_nhwc(xd), H.from_dev_nhwc(dd)
        out = torch.empty((N, h, w, cout), dtype=H.tdtype(wl), device="cuda")
        torch.cuda.synchronize()
        mod.forward(t, xd, out)
        did = mod.backward_delayed(t, delta_in=dd)
        mod.sync()
        ref = oracle.forward(1, t, x)
        ref_did, _, _ = oracle.backward_delayed(1, t, d, None, in_shape=x.shape)
        assert did == bool(ref_did) == (t >= 1)
        tol = parity.TOL[dtype]
        # (a batch norm over so few equal values divides by a variance that rounding decides)
        if N * h * w > 2:
            e = H.rel_err(H.from_dev_nhwc(out), ref)
            assert e < tol, (t, e)
            if did:
                e = H.rel_err(mod.get_grad(), oracle.get_grad(1))
                assert e < tol, (t, e)
        mod.update(t, 0.0)
        oracle.update(1, 0.0)
    mod.close()


SMALL = {"small_c16_5": ([(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)], 1, 5), "small_c16_24": ([(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)], 3, 24),
         "small_c32_7": ([(wk.BLOCK_BASIC, 32, 0, 32, 1, 0)], 5, 7), "small_c64_7": ([(wk.BLOCK_BASIC, 64, 0, 64, 1, 0)], 3, 7),
         "small_c32_to_64": ([(wk.BLOCK_BASIC, 32, 0, 64, 2, 1)], 5, 15), "small_c16_to_32": ([(wk.BLOCK_BASIC, 16, 0, 32, 2, 1)], 21, 28),
         "small_c128_6": ([(wk.BLOCK_BASIC, 128, 0, 128, 1, 0)], 2, 6)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(SMALL))
def test_small_launches(H, which, dtype, monkeypatch):
    monkeypatch.setitem(parity.SINGLE_BLOCKS, which, SMALL[which])
    parity.test_single_block_module(H, which, dtype)
