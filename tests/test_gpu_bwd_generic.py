"""Weight and input gradient of layers of the generic kernels: in one launch or two by the layer's size, operand type and company, counted;
and at size, against the oracle."""
import numpy as np
import pytest

import workloads as wk
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu
H = parity.H

# K of the pipeline, dtype, images of 28 x 28 x 16 (3 << 20 values lie between 250 and 251 of them), launches per layer
CASES = [(2, "f32", 250, 1), (2, "f32", 251, 2), (1, "f32", 251, 1), (2, "bf16", 251, 1), (2, "f32", 1, 1)]


@pytest.mark.parametrize("K,dtype,batch,launches", CASES)
def test_launches_of_a_generic_layer(K, dtype, batch, launches):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    print(f"case generic backward launches K={K} {dtype} batch={batch}", flush=True)
    hw, blocks = 28, [(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)]
    if K == 1:
        blocks = blocks + [(wk.BLOCK_HEAD, 16, 0, 0, 1, 0)]
    # (the second module of two without a head has a delay of none, the only module of one as well)
    mod = ddg.Module(make_desc(K, K, batch, (16, hw, hw), blocks, 10 if K == 1 else 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
    mod.set_params((wk.normal(3, 1, mod.param_count()) * 0.1 + 0.03).astype(np.float32))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((batch, hw, hw, 16), device="cuda").to(dt)
    labels = torch.zeros(batch, device="cuda", dtype=torch.int32)
    h, dx = torch.empty_like(x), torch.empty_like(x)
    torch.cuda.synchronize()
    mod.forward(0, x, None if K == 1 else h)
    mod.profile_enable(True)
    mod.backward_delayed(0, delta_in=None if K == 1 else x, labels=labels if K == 1 else None, delta_out=None if K == 1 else dx)
    mod.sync()
    ran = {kind: v[0] for kind, v in mod.profile_read().items() if v[0] and kind.startswith(("conv_wgrad", "conv_dgrad", "conv_bwd"))}
    # the block's second layer needs its input gradient; the first one does only where there is a module below
    both = 1 if K == 1 else 2
    alone = 2 - both                                     # layers with a weight gradient only
    want = {"conv_dgrad.generic": both}
    if launches == 2 or alone:
        want["conv_wgrad.generic"] = (both if launches == 2 else 0) + alone
    assert ran == want, ran
    mod.close()


AT_SIZE = {"generic_c16_28": ([(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)], 251, 28), "generic_c64_14": ([(wk.BLOCK_BASIC, 64, 0, 64, 1, 0)], 100, 14)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(AT_SIZE))
def test_generic_block_at_size(H, which, dtype, monkeypatch):
    monkeypatch.setitem(parity.SINGLE_BLOCKS, which, AT_SIZE[which])
    parity.test_single_block_module(H, which, dtype)
