"""The evaluation forward through the per-layer kernels, which serve what the many-layer kernel does not cover (and everything
under DDG_NO_FUSED_EVAL=1), and that kernel at a stem with stride 2: against the oracle with the same running estimates,
both entry points, the launches that ran counted."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu

STEM, BASIC, BOTTLENECK = wk.BLOCK_STEM, wk.BLOCK_BASIC, wk.BLOCK_BOTTLENECK
CIFAR = [(STEM, 3, 0, 16, 1, 0), (BASIC, 16, 0, 16, 1, 0), (BASIC, 16, 0, 32, 2, 1), (BASIC, 32, 0, 32, 1, 0),
         (BASIC, 32, 0, 64, 2, 1), (BASIC, 64, 0, 64, 1, 0)]
# blocks, height = width, batch, DDG_NO_FUSED_EVAL, is the many-layer kernel expected
CASES = {"switched_off": (CIFAR, 32, 3, True, False),
         "switched_off_ragged": (CIFAR, 11, 2, True, False),
         "128_channels": ([(BASIC, 32, 0, 64, 2, 1), (BASIC, 64, 0, 128, 2, 1), (BASIC, 128, 0, 128, 1, 0)], 16, 3, False, False),
         "wide_stem": ([(STEM, 3, 0, 32, 1, 0), (BASIC, 32, 0, 32, 1, 0)], 16, 2, False, False),
         "bottleneck": ([(BOTTLENECK, 64, 16, 64, 1, 0), (BOTTLENECK, 64, 32, 128, 2, 1)], 10, 3, False, False),
         "stem_stride_2": ([(STEM, 3, 0, 16, 2, 0), (BASIC, 16, 0, 16, 1, 0)], 32, 2, False, True),
         "stem_stride_2_odd": ([(STEM, 3, 0, 16, 2, 0), (BASIC, 16, 0, 32, 2, 1)], 13, 3, False, True),
         "stem_stride_2_large": ([(STEM, 4, 0, 16, 2, 0)], 90, 2, False, True)}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("which", sorted(CASES))
def test_evaluation_by_layers_matches_the_oracle(which, dtype, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    blocks, hw, N, off, fused = CASES[which]
    print(f"case evaluation by layers {which} {dtype}", flush=True)
    monkeypatch.setenv("DDG_NO_FUSED_EVAL", "1" if off else "0")
    cin, cout = blocks[0][1], blocks[-1][3]
    k = 1 if blocks[0][0] == STEM else 2
    mod = ddg.Module(make_desc(3, k, N, (cin, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(3, [blocks], N, (cin, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=k, store_bf16=(dtype == "bf16"))
    theta = (wk.normal(51, 1, mod.param_count()) * 0.1 + 0.03).astype(np.float32)
    mod.set_params(theta)
    oracle.set_params(k, theta.astype(np.float64))
    running = np.abs(wk.normal(53, 1, mod.running_count()) * 0.3).astype(np.float32) + np.float32(0.5)
    mod.set_running(running)
    oracle.set_running(k, running.astype(np.float64))

    class WL:
        pass
    wl = WL(); wl.dtype = dtype
    x = wk.normal(57, hw, N * cin * hw * hw).reshape(N, cin, hw, hw)
    xd = H.to_dev_nhwc(x, wl)
    if dtype == "bf16":
        x = H.from_dev_nhwc(xd)
    co, ho, wo = mod.out_shape()
    assert co == cout
    got = [torch.full((N, ho, wo, co), float("nan"), dtype=H.tdtype(wl), device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    mod.profile_enable(True)
    mod.forward_eval(xd, got[0])
    mod.forward_eval_static(xd, got[1])
    mod.sync()
    launches = {kind: v[0] for kind, v in mod.profile_read().items() if v[0]}
    assert ("eval_blocks" in launches) == fused, launches
    assert any(kind.startswith("conv_fprop") for kind in launches) == (not fused), launches
    mod.close()
    assert torch.equal(got[0], got[1])
    e = H.rel_err(H.from_dev_nhwc(got[0]), oracle.forward_eval(k, x))
    print(f"  rel err {e:.2e}", flush=True)
    # fp32: sums of up to 1152 products in another order; bf16: values that fall on the other side of a rounding boundary (2^-9)
    assert e <= (1e-4 if dtype == "f32" else 2e-2)
