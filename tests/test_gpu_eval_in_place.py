"""Evaluation of a module into memory that overlaps its input: the result is, bit for bit, that of the per-layer kernels or
(in place, image by image) of the many-layer kernel with separate buffers."""
import numpy as np
import pytest

import workloads as wk
from tests.eval_plan import launches, shapes

pytestmark = pytest.mark.gpu

IDENT = lambda c: (wk.BLOCK_BASIC, c, 0, c, 1, 0)
DOWN = (wk.BLOCK_BASIC, 16, 0, 32, 2, 1)
# blocks, height = width, offset of the output in images of the input; what it is there for
CASES = {"one_block": ([IDENT(16)], 24, 0),              # strips of rows whose halo a neighbour would overwrite
         "one_block_large": ([IDENT(16)], 44, 0),        # the same; bf16: an image just fits
         "one_block_strips": ([IDENT(16)], 52, 0),       # strips only, in bf16 too
         "two_blocks": ([IDENT(32)] * 2, 16, 0),         # bf16: whole images in place; fp32: two launches
         "down": ([DOWN, IDENT(32)], 16, 0),             # an image's output lies in another image's input
         "shifted": ([IDENT(64)] * 2, 8, 1)}             # by one image


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("which", sorted(CASES))
def test_output_may_overlap_the_input(which, dtype, static, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    blocks, hw, shift = CASES[which]
    print(f"case in place {which} {dtype} static={static}", flush=True)
    N, cin, cout = 64 if hw < 52 else 32, blocks[0][1], blocks[-1][3]     # (what the static scratch holds)
    ho = hw // blocks[0][4]
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    theta = None
    gen = torch.Generator(device="cuda"); gen.manual_seed(hw)
    x = torch.randn((N, hw, hw, cin), device="cuda", generator=gen).to(td)

    def evaluate(fused, overlap):
        nonlocal theta
        monkeypatch.setenv("DDG_NO_FUSED_EVAL", "0" if fused else "1")
        mod = ddg.Module(make_desc(3, 2, N, (cin, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
        if theta is None:
            theta = (wk.normal(41, hw, mod.param_count()) * 0.1 + 0.02).astype(np.float32)
        mod.set_params(theta)
        mem = torch.empty((N + shift) * hw * hw * cin, device="cuda", dtype=td)
        mem[:x.numel()] = x.flatten()
        off, n = shift * hw * hw * cin, N * ho * ho * cout
        out = mem[off:off + n] if overlap else torch.empty(n, device="cuda", dtype=td)
        torch.cuda.synchronize()
        mod.profile_enable(True)
        (mod.forward_eval_static if static else mod.forward_eval)(mem, out)
        mod.sync()
        res = out.clone()
        if fused:
            plan = launches(shapes(blocks), N, hw, dtype == "bf16")
            # with its output apart the plan; in place it, too, unless it is one launch that is not whole images to their own places
            want = len(plan) if not overlap or len(plan) > 1 else 1 if dtype == "bf16" and which in ("one_block", "one_block_large", "two_blocks") else 0
            assert mod.profile_read()["eval_blocks"][0] == want
            if which.startswith("one_block"):
                assert plan[0][1] > 1
        mod.close()
        return res
    layers, many, got = evaluate(False, False), evaluate(True, False), evaluate(True, True)
    assert torch.equal(got, layers) or torch.equal(got, many)
