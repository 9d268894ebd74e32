"""The optimizer step of a module above 2^20 parameters, which updates and repacks tile by tile: layers of one tile and of many,
with the narrowest and the widest tiles, next to layers that go value by value, and a classifier that ends the vector off a
16-byte boundary; bit for bit against a fresh module with the same weights, and against the optimizer's formula."""
import pytest

import workloads as wk
from tests import test_gpu_update_pack as small

pytestmark = pytest.mark.gpu

# 3-channel stem and 16-channel layers value by value, 16 -> 32 and 32 -> 64 at both stages' edges, taps as stored (the strided
# layers) and mirrored; 1x1 layers of 32 input channels (tiles narrower than 288 values) and of 2048 (several per row)
CASES = {"narrow": [(wk.BLOCK_STEM, 3, 0, 16, 1, 0), (wk.BLOCK_BASIC, 16, 0, 16, 1, 0), (wk.BLOCK_BASIC, 16, 0, 32, 2, 1)] +
         [(wk.BLOCK_BASIC, 32, 0, 64, 2, 1)] + [(wk.BLOCK_BASIC, 64, 0, 64, 1, 0)] * 14,
         "wide": [(wk.BLOCK_BOTTLENECK, 2048, 128, 2048, 1, 0), (wk.BLOCK_BOTTLENECK, 2048, 32, 2048, 1, 0),
                  (wk.BLOCK_BOTTLENECK, 2048, 128, 2048, 1, 0)]}


@pytest.mark.parametrize("opt", ["sgd", "adam"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(CASES))
def test_update_of_a_large_module(which, dtype, opt, monkeypatch):
    blocks = CASES[which]
    monkeypatch.setitem(small.CASES, which, (blocks, blocks[0][1], 16 if which == "narrow" else 4))
    small.test_update_repacks_every_operand(which, dtype, opt)


def test_large_module_with_a_classifier_of_ten():
    """4 x 2^18 weights and a 512 x 10 classifier: vectors whose length is no multiple of four, against NumPy."""
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    blocks = [(wk.BLOCK_BOTTLENECK, 512, 128, 512, 1, 0)] * 4 + [(wk.BLOCK_HEAD, 512, 0, 10, 1, 0)]
    print("case update classifier", flush=True)
    N, mu, wd, lr = 4, 0.9, 1e-3, 0.05
    mod = ddg.Module(make_desc(2, 2, N, (512, 4, 4), blocks, 10, ddg.DDG_BF16, mu, wd, 1e-5))
    w = (wk.normal(9, 1, mod.param_count()) * 0.05 + 0.02).astype(np.float32)
    assert w.size > 1 << 20 and w.size % 4 == 2
    mod.set_params(w)
    gen = torch.Generator(device="cuda"); gen.manual_seed(5)
    x = torch.randn((N, 4, 4, 512), device="cuda", generator=gen).to(torch.bfloat16)
    labels = torch.arange(N, device="cuda", dtype=torch.int32)
    dx, loss = torch.empty_like(x), torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    v, w = np.zeros(w.size), w.astype(np.float64)
    for t in range(3):
        mod.forward(t, x, None)
        mod.backward_delayed(t, labels=labels, delta_out=dx, loss_out=loss)
        mod.sync()
        v = mu * v + (mod.get_grad().astype(np.float64) + wd * w)
        w = w - lr * v
        mod.update(t, lr)
        mod.sync()
        got = mod.get_params().astype(np.float64)
        # three roundings of fp32 on each of v and w an update, the weights' own size the largest
        scale = np.abs(w).max() + lr * np.abs(v).max()
        assert np.abs(got - w).max() <= 6 * (t + 1) * 2.0 ** -24 * scale
    mod.close()
