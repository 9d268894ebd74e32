"""The evaluation kernel's identity blocks on images 512 / C pixels wide and high in bf16 (their own path: input rows shared by the
output rows they are taps of): one block and runs of three, one image and several, against the oracle; and infinities at
the corners, at the edges of a wave's rows and columns and inside, which must reach exactly the outputs that they are a tap of."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,batch", [(1, 1), (3, 2)])
@pytest.mark.parametrize("C", [16, 32, 64])
def test_square_identity_blocks(C, count, batch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    from tests.test_gpu_eval_inf import reached
    print(f"case square evaluation C={C} count={count} batch={batch}", flush=True)
    hw, block = 512 // C, (wk.BLOCK_BASIC, C, 0, C, 1, 0)
    blocks = [block] * count
    mod = ddg.Module(make_desc(3, 2, batch, (C, hw, hw), blocks, 0, ddg.DDG_BF16, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(3, [blocks], batch, (C, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=2, store_bf16=True)
    theta = (wk.normal(51, C, mod.param_count()) * 0.1 + 0.03).astype(np.float32)
    running = np.abs(wk.normal(53, C, mod.running_count()) * 0.3).astype(np.float32) + np.float32(0.5)

    class WL:
        dtype = "bf16"
    xd = H.to_dev_nhwc(wk.normal(57, hw, batch * C * hw * hw).reshape(batch, C, hw, hw), WL)

    def forward(th, x):
        mod.set_params(th)
        mod.set_running(running)
        h = x.clone()             # (in place an image is never cut into strips)
        torch.cuda.synchronize()
        mod.forward_eval_static(h, h)
        mod.sync()
        return h

    oracle.set_params(2, theta.astype(np.float64))
    oracle.set_running(2, running.astype(np.float64))
    e = H.rel_err(H.from_dev_nhwc(forward(theta, xd)), oracle.forward_eval(2, H.from_dev_nhwc(xd)))
    print(f"  rel err {e:.2e}", flush=True)
    assert e <= 2e-2       # both sides round at the same points; values on the other side of a rounding boundary differ by 2^-9 of themselves
    if count == 1:
        theta = np.abs(theta) * np.float32(0.1) + np.float32(0.01)
        mask = np.zeros((batch, hw, hw), bool)
        for h, w in ((0, 0), (hw - 1, hw - 1), (hw // 2 - 1, hw // 2), (hw // 4, 0), (0, hw - 1)):
            mask[0, h, w] = True
        xf = xd.abs()
        xi = xf.clone()
        xi[torch.from_numpy(mask).to("cuda")] = torch.tensor([float("inf")] + [1.0] * (C - 1), device="cuda").to(torch.bfloat16)
        xf = torch.where(torch.isinf(xi), torch.ones_like(xi), xi)
        got, finite = (forward(theta, v).float().cpu().numpy() for v in (xi, xf))
        want = np.repeat(reached(mask, block)[..., None], C, axis=3)
        assert want.any() and not want.all()
        assert np.array_equal(np.isposinf(got), want)
        assert np.isfinite(finite).all()
        assert np.array_equal(got[~want], finite[~want])
    mod.close()
