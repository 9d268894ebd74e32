"""The forward pass that reads its input where it is and keeps a copy with its last launch: the output written over the input, or
over a part of it, gives the bits that separate buffers give, for the backward pass too."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("place", ["apart", "over", "shifted"])
@pytest.mark.parametrize("dtype,batch,hw", [("bf16", 3, 8), ("f32", 1, 5), ("bf16", 1, 5)])
def test_output_over_input(place, dtype, batch, hw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    print(f"case forward tail {place} {dtype} batch={batch} hw={hw}", flush=True)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    n = batch * hw * hw * 16

    def run(where):
        m = ddg.Module(make_desc(2, 1, batch, (16, hw, hw), [(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)] * 2, 0,
                                 ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
        m.set_params((wk.normal(3, 1, m.param_count()) * 0.1 + 0.05).astype(np.float32))
        out = []
        for t in range(4):
            buf = torch.zeros(3 * n, device="cuda", dtype=td)
            buf[:n] = torch.from_numpy(wk.normal(5, t, n).astype(np.float32)).to("cuda").to(td)
            o = {"apart": 2 * n, "over": 0, "shifted": n - 16}[where]
            x, h = buf[:n], buf[o:o + n]
            d = torch.from_numpy(wk.normal(7, t, n).astype(np.float32)).to("cuda").to(td)
            torch.cuda.synchronize()
            m.forward(t, x, h)
            did = m.backward_delayed(t, delta_in=d)
            m.sync()
            out += [h.float().cpu().numpy().copy()] + ([m.get_grad()] if did else [])
            m.update(t, 0.01)
        m.sync()
        m.close()
        return out
    for a, b in zip(run(place), run("apart")):
        assert np.isfinite(a).all() and np.array_equal(a, b)
