"""The wide weight-gradient kernel on its own (called through the library's own launcher): its error against 64-bit sums stays
within the roundings it makes, whatever the number of pixels in a slice; infinities come out as infinities."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

NAMES = ["N", "H", "W", "Cin", "Cout", "R", "splits"]


class Layer(C.Structure):      # WgradWideLayer
    _fields_ = [(n, C.c_void_p) for n in ("x", "dz", "scale", "shift", "partial")] + [(n, C.c_int) for n in NAMES]


def run(x, dz, *sizes):
    import torch
    from paper_1804_10574_amd.ddg import load_library
    N, H, W, Cin, Cout, R, splits = sizes
    assert x.shape == (N * H * W, Cin) and dz.shape == (N * H * W, Cout) and splits <= (N * H * W + 63) // 64
    part = torch.full((splits, Cout, R * R * Cin), 7.0, device="cuda")
    torch.cuda.synchronize()
    layer = Layer(x.data_ptr(), dz.data_ptr(), None, None, part.data_ptr(), *sizes)
    launch = load_library()._ZN3ddg17wgrad_wide_launchEPKNS_14WgradWideLayerEiP12ihipStream_t
    assert launch(C.byref(layer), C.c_int(1), C.c_void_p(None)) == 0
    torch.cuda.synchronize()
    s = part[0].clone()                                  # rows in order
    for k in range(1, splits):
        s += part[k]
    return s


def exact(x, dz, N, H, W, R):
    import torch
    xd, zt = x.double().view(N, H, W, -1), dz.double().t().contiguous()
    if R == 1:
        return zt @ xd.reshape(N * H * W, -1)
    pad = torch.nn.functional.pad(xd, (0, 0, 1, 1, 1, 1))
    return torch.cat([zt @ pad[:, t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(N * H * W, -1) for t in range(9)], 1)


# (pixels as N x hw x hw, channels, kernel, slices): long slices of the sizes that bottleneck modules have, and steps of a slice on both
# sides of the lines at 2 and 8
CASES = [(32, 14, 256, 1024, 1, 2), (32, 14, 256, 256, 3, 2), (64, 28, 512, 128, 1, 16), (64, 7, 512, 512, 3, 1), (1, 14, 256, 256, 3, 2),
         (3, 8, 128, 128, 3, 1), (2, 8, 256, 128, 1, 1), (8, 8, 128, 256, 1, 1), (9, 8, 128, 256, 1, 1), (1, 5, 128, 128, 3, 1)]


@pytest.mark.parametrize("N,hw,Cin,Cout,R,splits", CASES)
def test_error_against_64_bits(N, hw, Cin, Cout, R, splits):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    gen = torch.Generator(device="cuda"); gen.manual_seed(3)
    M = N * hw * hw
    x = torch.randn((M, Cin), device="cuda", generator=gen).relu_().bfloat16()
    dz = torch.randn((M, Cout), device="cuda", generator=gen).bfloat16()
    ref = exact(x, dz, N, hw, hw, R)
    err = float((run(x, dz, N, hw, hw, Cin, Cout, R, splits).double() - ref).norm() / ref.norm())
    # A rounding to nearest of a partial sum p is off by 2^-24 |p| / sqrt(3) at most (2-norm over many). The squares of the partial
    # sums that are rounded, as shares of the result's: a chain of n matrix instructions of 16 pixels (1 + .. + n)/n of its own
    # share, with n = 8 (two steps); an addition of two accumulators whose rest is kept, 1 at most for the rest; the last
    # addition 1; the slices in order (2 + .. + splits)/splits.
    shares = 4.5 + 1 + 1 + sum(range(2, splits + 1)) / splits
    print(f"case wide wgrad error {N}x{hw}x{hw} {Cin}-{Cout} {R}x{R}: {err:.2e}", flush=True)
    assert err <= 2.0 ** -24 * (shares / 3) ** 0.5


@pytest.mark.parametrize("N", [1, 3, 20])            # slices of 2, 5 and 32 steps
def test_infinities_stay_infinities(N):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    gen = torch.Generator(device="cuda"); gen.manual_seed(4)
    M = N * 100
    x = torch.randn((M, 128), device="cuda", generator=gen).abs().add_(0.5).bfloat16()
    dz = torch.randn((M, 128), device="cuda", generator=gen).bfloat16()
    dz[M // 2, 5] = float("inf")                         # one channel with an infinity, one that overflows, one that is no number
    dz[M // 3:M // 3 + 8, 77] = -3e38
    dz[M - 1, 9] = float("nan")
    got, ref = run(x, dz, N, 10, 10, 128, 128, 1, 1), exact(x, dz, N, 10, 10, 1)
    assert bool((got[5] == float("inf")).all()) and bool((got[77] == float("-inf")).all()) and bool(got[9].isnan().all())
    rest = [c for c in range(128) if c not in (5, 77, 9)]
    assert float((got[rest].double() - ref[rest]).norm() / ref[rest].norm()) <= 2.0 ** -24 * (6.5 / 3) ** 0.5
