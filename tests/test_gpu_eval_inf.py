"""Infinite activations in the evaluation kernel that keeps activations in LDS: an infinity in the input makes every output
infinite that it reaches through positive weights, and no other output changes by a bit. The contraction of 16 channels
(bf16) and of the stem ends inside a k-step, whose lanes past the last tap multiply zero weights: 0 * inf there
would be NaN, and 0 after the ReLU."""
import numpy as np
import pytest

import workloads as wk
from tests.eval_plan import launches, shapes

pytestmark = pytest.mark.gpu

BLOCKS = {"stem": (wk.BLOCK_STEM, 3, 0, 16, 1, 0), "stem_s2": (wk.BLOCK_STEM, 3, 0, 16, 2, 0),
          "identity16": (wk.BLOCK_BASIC, 16, 0, 16, 1, 0), "down16": (wk.BLOCK_BASIC, 16, 0, 32, 2, 1),
          "identity32": (wk.BLOCK_BASIC, 32, 0, 32, 1, 0)}


def reached(mask, block):
    """Output pixels that a marked input pixel reaches ([n][h][w], booleans)."""
    import torch
    import torch.nn.functional as F
    kind, stride = block[0], block[4]

    def conv(m, s):
        return F.conv2d(m[:, None].float(), torch.ones(1, 1, 3, 3), stride=s, padding=1)[:, 0] > 0
    m = torch.from_numpy(mask)
    if kind == wk.BLOCK_STEM:
        return conv(m, stride).numpy()
    return (conv(conv(m, stride), 1) | m[:, ::stride, ::stride]).numpy()


# bf16: 256 images: whole (33: more pixels than a wave's registers hold; 32 channels of it exceed LDS); 64: strips of several rows;
# two: strips of a row or two, and whole images where the map is small; fp32: strips
@pytest.mark.parametrize("hw,N", [(10, 2), (33, 2), (44, 2), (44, 64), (52, 64), (10, 256), (33, 256)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("which", sorted(BLOCKS))
def test_an_infinity_reaches_what_it_should(which, dtype, hw, N):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    print(f"case infinity {which} {dtype} hw={hw} N={N}", flush=True)
    block = BLOCKS[which]
    cin, cout, stride = block[1], block[3], block[4]
    strips = launches(shapes([block]), N, hw, dtype == "bf16")[0][1]
    if dtype == "bf16" and (N > 2 or hw > 10):
        assert (strips == 1) == (N == 256 and (which, hw) != ("identity32", 33))
    ho = (hw - 1) // stride + 1
    mod = ddg.Module(make_desc(2, 1, N, (cin, hw, hw), [block], 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
    theta = np.abs(wk.normal(31, 1, mod.param_count()) * 0.05).astype(np.float32) + np.float32(0.01)
    mod.set_params(theta)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.from_numpy(np.abs(wk.normal(37, hw, N * hw * hw * cin)).reshape(N, hw, hw, cin).astype(np.float32)).to("cuda").to(td)
    mask = np.zeros((N, hw, hw), bool)
    for n, h, w in ((0, 0, 0), (0, 6, 5), (1, 3, 7), (1, hw - 1, hw - 1)):      # (odd positions: tap 0 of stride 2)
        mask[n, h, w] = True
    xi = x.clone()
    xi[torch.from_numpy(mask).to("cuda")] = torch.tensor([float("inf")] + [1.0] * (cin - 1), device="cuda").to(td)
    xf = torch.where(torch.isinf(xi), torch.ones_like(xi), xi)
    out = {}
    mod.profile_enable(True)
    for name, inp in (("inf", xi), ("finite", xf)):
        h = torch.empty((N, ho, ho, cout), dtype=td, device="cuda")
        torch.cuda.synchronize()
        mod.forward_eval(inp, h)
        mod.sync()
        out[name] = h.float().cpu().numpy()
    assert mod.profile_read()["eval_blocks"][0] > 0
    mod.close()
    want = np.repeat(reached(mask, block)[..., None], cout, axis=3)
    assert want.any() and not want.all()
    assert np.array_equal(np.isposinf(out["inf"]), want)
    assert np.isfinite(out["finite"]).all()
    assert np.array_equal(out["inf"][~want], out["finite"][~want])
