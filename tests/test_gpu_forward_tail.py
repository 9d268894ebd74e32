"""The forward pass that reads its input where it is and keeps a copy with its last launch: the output written over the input, or
over a part of it, and an input on no more than a 16-byte boundary give the bits that separate buffers give, for the backward
pass too; three-channel inputs whose byte count has a remainder, and one above 4 MiB, which is copied first."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu

CASES = [("bf16", 3, 8, 16), ("f32", 1, 5, 16), ("bf16", 1, 5, 16), ("bf16", 1, 5, 3), ("f32", 3, 7, 3), ("bf16", 129, 32, 16)]


@pytest.mark.parametrize("place", ["over", "shifted", "offset"])
@pytest.mark.parametrize("dtype,batch,hw,cin", CASES)
def test_input_read_in_place(place, dtype, batch, hw, cin):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    print(f"case forward tail {place} {dtype} batch={batch} hw={hw} cin={cin}", flush=True)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    n, ni = batch * hw * hw * 16, batch * hw * hw * cin
    unit = 8 if dtype == "bf16" else 4                   # elements of 16 bytes
    blocks = [(wk.BLOCK_STEM, 3, 0, 16, 1, 0)] * (cin == 3) + [(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)] * 2
    inputs = [torch.from_numpy(wk.normal(5, t, ni).astype(np.float32)).to("cuda").to(td) for t in range(4)]
    deltas = [torch.from_numpy(wk.normal(7, t, n).astype(np.float32)).to("cuda").to(td) for t in range(4)]

    def run(where):
        m = ddg.Module(make_desc(2, 1, batch, (cin, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32,
                                 0.9, 0.0, 1e-5))
        m.set_params((wk.normal(3, 1, m.param_count()) * 0.1 + 0.05).astype(np.float32))
        out = []
        for t in range(4):
            buf = torch.zeros(3 * n, device="cuda", dtype=td)
            i = unit if where == "offset" else 0
            o = {"apart": 2 * n, "over": 0, "shifted": (ni - 1) // unit * unit, "offset": 2 * n}[where]
            x, h = buf[i:i + ni], buf[o:o + n]
            x.copy_(inputs[t])
            torch.cuda.synchronize()
            m.forward(t, x, h)
            did = m.backward_delayed(t, delta_in=deltas[t])
            m.sync()
            out += [h.float().cpu().numpy().copy()] + ([m.get_grad()] if did else [])
            m.update(t, 0.01)
        m.sync()
        m.close()
        return out
    for a, b in zip(run(place), run("apart")):
        assert np.isfinite(a).all() and np.array_equal(a, b)
