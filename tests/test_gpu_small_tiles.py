"""Generic bf16 convolutions of few waves run in smaller tiles. Outputs and statistics rows are those of the wide tiles bit for bit: what a thread adds in
fp32 does not depend on how the channels are shared out."""
import pytest

from tests import launchers as L

pytestmark = pytest.mark.gpu

# input channels, output channels, stride, images, size: one wave and just below 512 waves of wide tiles, ragged pixels, one to eight channel blocks
LAYERS = [(16, 16, 1, 1, 3), (16, 16, 1, 5, 28), (16, 32, 2, 37, 32), (32, 32, 1, 8, 14), (32, 64, 2, 37, 16), (64, 64, 1, 8, 7), (64, 64, 1, 1, 1),
          (48, 48, 1, 3, 9), (128, 128, 1, 2, 6), (16, 16, 1, 41, 28), (16, 16, 1, 42, 28)]


@pytest.mark.parametrize("cin,cout,stride,N,hw", LAYERS)
@pytest.mark.parametrize("dgrad", [0, 1])
def test_same_bits_as_wide_tiles(cin, cout, stride, N, hw, dgrad):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    if dgrad and stride == 2:
        pytest.skip("not a launch of this kernel")
    print(f"case small tiles {cin}-{cout}/{stride} {N}x{hw}x{hw} dgrad {dgrad}", flush=True)
    gen = torch.Generator(device="cuda"); gen.manual_seed(cin + N)
    f = dict(device="cuda", generator=gen)
    results, shapes = [], []
    x = w = wp = None
    for wide in (False, True):
        a, n = L.conv_args(N, hw, hw, cin, cout, stride, L.BF16, dgrad)
        if wide:
            ocb = a.OC // 16
            a.nb, a.mb = (4, 2) if ocb % 4 == 0 else (2, 2) if ocb % 2 == 0 else (1, 4)
            a.grid_x = min(((a.M + 16 * a.mb - 1) // (16 * a.mb) + 3) // 4, 512 // (ocb // a.nb))
        if x is None:
            x = torch.randn((N, a.IH, a.IW, a.IC), **f).bfloat16()
            w = torch.randn((cout, cin, 3, 3), **f) * (2 / (9 * cin)) ** 0.5
            wp = L.pack(w, a, n)
        out = torch.full((a.M, a.OC), 7.0, device="cuda", dtype=torch.bfloat16)
        stat = torch.full((a.grid_x, 2, a.OC), 9.0, device="cuda")
        a.in_, a.wpack, a.out, a.stat = x.data_ptr(), wp.data_ptr(), out.data_ptr(), None if dgrad else stat.data_ptr()
        torch.cuda.synchronize()
        L.conv(a)
        torch.cuda.synchronize()
        results.append((out, stat if not dgrad else out))
        shapes.append((a.mb, a.nb, a.grid_x))
    assert dgrad or shapes[0][::2] == shapes[1][::2], shapes
    for small, wide in zip(*results):
        assert torch.equal(small, wide), shapes
