"""Rows of partial weight gradients: minibatches with a tile a row and with tiles that are shared out unevenly, against the oracle; and more than 64 rows a layer, where the pipeline's sums-update-repack launch has twice as many of them
in flight, bit for bit against the launch that only adds."""
import pytest

import workloads as wk
from workloads.configs import custom_cifar
from tests import test_gpu_parity as parity
from tests import test_gpu_shared_launches as shared

pytestmark = pytest.mark.gpu
H = parity.H

IDENT = lambda c: [(wk.BLOCK_BASIC, c, 0, c, 1, 0)]
# channels, images, size: tiles of 8 rows, for at most 128 / 64 / 16 partial tiles
ROWS = {f"c{c}_n{n}": (IDENT(c), n, hw) for c, hw, ns in ((16, 32, (1, 33)), (32, 16, (1, 33)), (64, 8, (1, 2, 4, 49))) for n in ns}


@pytest.mark.parametrize("which", sorted(ROWS))
def test_shares_of_tiles(H, which, monkeypatch):
    monkeypatch.setitem(parity.SINGLE_BLOCKS, which, ROWS[which])
    parity.test_single_block_module(H, which, "bf16")


# 16 channels at 32x32 are four tiles an image: fp32 rows 64, 68, 80, 128; bf16 128, 128
@pytest.mark.parametrize("dtype,batch", [("f32", 16), ("f32", 17), ("f32", 20), ("f32", 33), ("bf16", 33), ("bf16", 49)])
def test_rows_in_flight(H, dtype, batch, monkeypatch):
    name = f"rows_{batch}"
    monkeypatch.setitem(shared.CASES, name, lambda d: custom_cifar(1, [2], batch=batch, num_classes=10, hw=32, dtype=d, name=name))
    shared.test_pipeline_update_is_the_call_by_call_update(H, name, dtype, "sgd")
