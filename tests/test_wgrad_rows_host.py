"""How many partial tiles the tiled bf16 weight gradients write (host code, no GPU): a tile of the image a row until the rows run out. Two or
three tiles a row are shorter at small minibatches, but an accumulator that runs on over them rounds more often: against 64-bit sums the gradients of 64
channels were off by 4.4e-8 with a tile a row and by 5.3e-8 with three (three images), 6.1e-8 and 6.7e-8 (13), 7.9e-8 and 8.2e-8 (50)."""
import pytest

from paper_1804_10574_amd.ddg import load_library


@pytest.mark.parametrize("c,hw,most", [(16, 32, 128), (32, 16, 64), (64, 8, 16)])
def test_a_tile_a_row(c, hw, most):
    rows = load_library()._ZN3ddg16wgrad_tiled_rowsEiiiiiiii
    for n in range(1, 130):
        assert rows(n, hw, hw, c, c, 3, 1, 1) == min(most, n * hw // 8)
