"""The optimizer step that repacks the operands as it goes: after three updates a module computes, bit for bit, what a fresh
module does that was given the same weights (every packed operand is where the convolutions look for it, padding
included), and the weights are the optimizer's formula applied to the gradients."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu

# blocks, input channels, size, what is there: a 3-channel stem (padded contraction), LDS-tiled layers (mirrored taps), a stage
# change (taps as stored, projection); a wide block above the line of 2^20 parameters (the launch that goes tile by tile), one below
CASES = {"cifar": ([(wk.BLOCK_STEM, 3, 0, 16, 1, 0), (wk.BLOCK_BASIC, 16, 0, 16, 1, 0), (wk.BLOCK_BASIC, 16, 0, 32, 2, 1)], 3, 32),
         "wide_1114k": ([(wk.BLOCK_BOTTLENECK, 1024, 256, 1024, 1, 0)], 1024, 4),
         "wide_280k": ([(wk.BLOCK_BOTTLENECK, 512, 128, 512, 1, 0)], 512, 4)}


@pytest.mark.parametrize("opt", ["sgd", "adam"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(CASES))
def test_update_repacks_every_operand(which, dtype, opt):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    blocks, c, hw = CASES[which]
    print(f"case update {which} {dtype} {opt}", flush=True)
    N, mu, wd, lr = 4, 0.9, 1e-3, 0.05 if opt == "sgd" else 1e-2
    first = c == 3
    K, k = (2, 1) if first else (2, 2)
    cout, down = blocks[-1][3], int(np.prod([b[4] for b in blocks]))
    ho = hw // down

    def module():
        m = ddg.Module(make_desc(K, k, N, (c, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, mu, wd, 1e-5))
        if opt == "adam":
            m.set_optimizer(ddg.DDG_OPT_ADAM)
        return m
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda"); gen.manual_seed(5)
    mod = module()
    w = (wk.normal(9, 1, mod.param_count()) * 0.05 + 0.02).astype(np.float32)
    mod.set_params(w)
    x = [torch.randn((N, hw, hw, c), device="cuda", generator=gen).to(td) for _ in range(2)]
    delta = [torch.randn((N, ho, ho, cout), device="cuda", generator=gen).to(td) for _ in range(2)]
    h, dx = torch.empty_like(delta[0]), None if first else torch.empty_like(x[0])
    torch.cuda.synchronize()
    v, m2, n = np.zeros(w.size), np.zeros(w.size), 0
    w = w.astype(np.float64)
    for t in range(4):
        mod.forward(t, x[t % 2], h)
        did = mod.backward_delayed(t, delta_in=delta[t % 2], delta_out=dx)
        mod.sync()
        if did:
            g = mod.get_grad().astype(np.float64) + wd * w
            n += 1
            if opt == "sgd":
                v = mu * v + g
                w = w - lr * v
            else:
                b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
                v, m2 = b1 * v + (1 - b1) * g, b2 * m2 + (1 - b2) * g * g
                w = w - lr * (v / (1 - b1 ** n)) / (np.sqrt(m2 / (1 - b2 ** n)) + 1e-8)
        mod.update(t, lr)
        mod.sync()
        got = mod.get_params()
        # fp32 rounding of weight and step. Adam divides the gradient by its own size: where gradient and weight decay
        # cancel to within rounding (2^-24 of either; a fraction of about 1e-4 of the weights for a relative 1e-4 of
        # the step) the quotient has no digits left
        close = np.isclose(got, w, rtol=1e-5, atol=lr * 1e-4 if opt == "adam" else 1e-6)
        assert close.all() if opt == "sgd" else close.mean() > 0.999
        w = got.astype(np.float64)
    fresh = module()
    fresh.set_params(mod.get_params())
    hf, dxf = torch.empty_like(h), None if first else torch.empty_like(dx)
    torch.cuda.synchronize()
    # the running module's next forward and backward use operands that only updates have written
    mod.forward(4, x[0], h)
    mod.backward_delayed(4, delta_in=delta[0], delta_out=dx)
    mod.sync()
    start = 0 if K == k else 1          # (with a delay of 1 the first backward of the fresh module comes an iteration later)
    for t in range(start + 1):
        fresh.forward(t, x[0] if t == start else x[1], hf)
        fresh.backward_delayed(t, delta_in=delta[0], delta_out=dxf)
        if t < start:
            fresh.update(t, 0.0)
    fresh.sync()
    assert torch.equal(h, hf)
    if dx is not None:
        assert torch.equal(dx, dxf)
    mod.close(); fresh.close()
