"""Blocks whose first layer forms the block's input while it loads (the output of the block before): pixels on both sides of a
tile of 64, both tile shapes (128 and 256 output channels), the fewest and the most input channels, statistics of as many rows as
one trip of 16 takes and of more, with and without rests, in paired forward passes; against the oracle, the normalising launches
counted."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu

CASES = [(1, 3, 256, 128, 3),      # 9 pixels, four chunks of channels (the fewest)
         (1, 8, 512, 256, 3),      # 64 pixels: one tile exactly
         (5, 5, 2048, 128, 3),     # 125 pixels, the most input channels: the largest table of scales
         (1, 13, 512, 256, 3),     # 169 pixels: last tile of 41
         (13, 5, 1024, 256, 3),    # 325 pixels: last tile of 5
         (10, 14, 512, 128, 2),    # 1960 pixels: 31 rows of a tile each, one fewer than the most sums
         (20, 8, 2048, 128, 2)]    # 1280 pixels: rows of two and three tiles, with rests: 20 for one minibatch, 2*7 for two


@pytest.mark.parametrize("batch,hw,c,cmid,blocks", CASES)
def test_first_layer_forms_its_input(batch, hw, c, cmid, blocks):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    print(f"case formed inputs batch={batch} hw={hw} {c}-{cmid}-{c}", flush=True)
    net, shape = [(wk.BLOCK_BOTTLENECK, c, cmid, c, 1, 0)] * blocks, (batch, c, hw, hw)
    mod = ddg.Module(make_desc(4, 2, batch, (c, hw, hw), net, 0, ddg.DDG_BF16, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(4, [net], batch, (c, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=2, store_bf16=True)
    theta = (wk.normal(31, 1, oracle.param_count(2)) * 0.05 + 0.02).astype(np.float32)
    oracle.set_params(2, theta.astype(np.float64))
    mod.set_params(theta)

    class WL:
        dtype = "bf16"
    keep = []
    for t in range(4):
        hd = H.to_dev_nhwc(wk.normal(33, t, int(np.prod(shape))).reshape(shape), WL)
        dd = H.to_dev_nhwc(wk.normal(37, t, int(np.prod(shape))).reshape(shape), WL)
        h_out, d_out = torch.empty_like(hd), torch.zeros_like(hd)
        keep += [hd, dd, h_out, d_out]
        torch.cuda.synchronize()
        mod.profile_reset()
        mod.profile_enable(True)
        mod.forward(t, hd, h_out)
        mod.profile_enable(False)
        # the last block's output only; the others' are formed by the block behind
        assert mod.profile_read()["bn_apply"][0] == 1
        did = mod.backward_delayed(t, delta_in=dd, delta_out=d_out)
        mod.sync()
        ref_h = oracle.forward(2, t, H.from_dev_nhwc(hd))
        ref_did, ref_dx, _ = oracle.backward_delayed(2, t, H.from_dev_nhwc(dd), None, in_shape=shape)
        assert did == bool(ref_did)
        e_h = H.rel_err(H.from_dev_nhwc(h_out), ref_h)
        print(f"  t={t} h {e_h:.2e}", flush=True)
        # both sides round at the same points: a value on the other side of a rounding boundary is off by 2^-8 of itself at
        # most, and each of the 9 layers behind the input turns at most all of them: sqrt(9) * 2^-8
        assert e_h <= 3 * 2.0 ** -8
        if did:
            e_d, e_g = H.rel_err(H.from_dev_nhwc(d_out), ref_dx), H.rel_err(mod.get_grad(), oracle.get_grad(2))
            print(f"      dx {e_d:.2e} grad {e_g:.2e}", flush=True)
            # ReLU decisions near zero, a fraction f < 1e-3 of each of 9: sqrt(9 f)
            assert e_d <= 9.5e-2 and e_g <= 9.5e-2
        # (rate 0: gradients of the two sides differ by the flipped decisions above, up to 9.5e-2 of themselves, and weights
        # moved by them would no longer be the same inputs)
        mod.update(t, 0.0)
        oracle.update(2, 0.0)
    mod.close()
