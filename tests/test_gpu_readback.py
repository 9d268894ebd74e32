"""Weights read back through the ring of pinned slots: sizes below and above the line from which it is used,
with a ragged last piece, twice in a row and from two threads at once."""
import threading

import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu


# parameters: 16.0K (one piece), 1.12 M (below 8 MiB), 2.23 M and 4.46 M (above, ragged, more pieces than slots)
@pytest.mark.parametrize("c,mid,blocks", [(32, 32, 1), (1024, 256, 1), (1024, 256, 2), (1024, 256, 4)])
def test_weights_come_back_bit_for_bit(c, mid, blocks):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    print(f"case readback c={c} blocks={blocks}", flush=True)
    mod = ddg.Module(make_desc(3, 2, 1, (c, 4, 4), [(wk.BLOCK_BOTTLENECK, c, mid, c, 1, 0)] * blocks, 0, ddg.DDG_BF16,
                               0.9, 0.0, 1e-5))
    theta = wk.normal(3, blocks, mod.param_count()).astype(np.float32)
    mod.set_params(theta)
    for _ in range(2):
        assert np.array_equal(mod.get_params(), theta)
    assert not mod.get_velocity().any()
    got = [None, None]

    def read(i):
        got[i] = mod.get_params()
    threads = [threading.Thread(target=read, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(np.array_equal(g, theta) for g in got)
    mod.close()
