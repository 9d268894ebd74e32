"""Evaluation with 16 bytes between the pixels in LDS (bf16), whole images and strips, every stage of a network: against the
oracle, the first and the last image of the minibatch."""
import numpy as np
import pytest

import workloads as wk
from tests.eval_plan import launches, shapes

pytestmark = pytest.mark.gpu

STEM, DOWN = (wk.BLOCK_STEM, 3, 0, 16, 1, 0), lambda c: (wk.BLOCK_BASIC, c, 0, 2 * c, 2, 1)
IDENT = lambda c: (wk.BLOCK_BASIC, c, 0, c, 1, 0)
# blocks, height = width, images, whole images
CASES = [([IDENT(32)] * 2, 28, 200, True), ([IDENT(64)] * 2, 18, 256, True), ([DOWN(32), IDENT(64)], 24, 256, True),
         ([STEM, IDENT(16), DOWN(16), IDENT(32), DOWN(32), IDENT(64)], 33, 64, True), ([IDENT(32)], 38, 64, False), ([IDENT(64)], 24, 256, False)]


@pytest.mark.parametrize("blocks,hw,batch,whole", CASES)
def test_narrow_pitch_matches_the_oracle(blocks, hw, batch, whole):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    print(f"case narrow pitch {len(blocks)} blocks from {blocks[0][1]} channels hw={hw} batch={batch}", flush=True)
    assert [(strips == 1, gap) for _, strips, gap, _ in launches(shapes(blocks), batch, hw)] == [(whole, 16)]
    cin, k = blocks[0][1], 1 if blocks[0] is STEM else 2
    mod = ddg.Module(make_desc(3, k, batch, (cin, hw, hw), blocks, 0, ddg.DDG_BF16, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(3, [blocks], 2, (cin, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=k, store_bf16=True)
    theta = (wk.normal(51, hw, mod.param_count()) * 0.1 + 0.03).astype(np.float32)
    running = np.abs(wk.normal(53, hw, mod.running_count()) * 0.3).astype(np.float32) + np.float32(0.5)
    mod.set_params(theta)
    mod.set_running(running)
    oracle.set_params(k, theta.astype(np.float64))
    oracle.set_running(k, running.astype(np.float64))

    class WL:
        dtype = "bf16"
    x = H.to_dev_nhwc(wk.normal(57, hw, batch * cin * hw * hw).reshape(batch, cin, hw, hw), WL)
    co, ho, wo = mod.out_shape()
    h = torch.full((batch, ho, wo, co), float("nan"), device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    mod.profile_enable(True)
    mod.forward_eval(x, h)
    ran = {kind: v[0] for kind, v in mod.profile_read().items() if v[0]}
    assert ran == {"eval_blocks": 1}, ran
    mod.close()
    ends = [0, batch - 1]
    e = H.rel_err(H.from_dev_nhwc(h[ends]), oracle.forward_eval(k, H.from_dev_nhwc(x[ends])))
    print(f"  rel err {e:.2e}", flush=True)
    assert e <= 2e-2       # both sides round at the same points; values on the other side of a rounding boundary differ by 2^-9 of themselves
    assert torch.isfinite(h).all()
