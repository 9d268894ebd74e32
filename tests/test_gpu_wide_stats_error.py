"""The statistics rows of the 1x1 kernel for few contraction channels, called through the library's own launcher: however many
pixels a row stands for, the sums are no further from 64-bit sums than with a row per 64 pixels."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


class Below(C.Structure):      # ConvStat
    _fields_ = [("mode", C.c_int)] + [(n, C.c_void_p) for n in ("partial", "mask", "mscale", "mshift", "z", "zmean", "zinvstd")]


class Second(C.Structure):     # ConvWideSecond
    _fields_ = [(n, C.c_void_p) for n in ("in_", "out", "stat", "scale", "shift")]


def former(g, f=None):
    """Sums over the pixels (rows) of g, or of g*f, with a row per 64 pixels: fp32 sums of pixels p and p + 32, those 32 in order, the rows in
    64 bits."""
    import torch
    M, n = g.shape[0], g.shape[1]
    pad = (0, 0, 0, -M % 64)
    v = torch.nn.functional.pad(g, pad).view(-1, 2, 32, n)
    if f is None:
        p = v[:, 0] + v[:, 1]
    else:
        w = torch.nn.functional.pad(f, pad).view(-1, 2, 32, n)
        p = (v[:, 1].double() * w[:, 1].double() + (v[:, 0] * w[:, 0]).double()).float()       # (one rounding each)
    s = torch.zeros_like(p[:, 0])
    for r in range(32):
        s += p[:, r]
    return s.double().sum(0)


# pixels as N x hw x hw, channels, minibatches of the launch: a tile a group (the last one ragged), 4, 7 and 8 tiles a group, 9 and more
# (sums that move between tiles), one group of many tiles
CASES = [(5, 10, 128, 512, 1), (32, 14, 256, 1024, 1), (32, 14, 256, 1024, 2), (16, 16, 256, 2048, 2), (43, 14, 256, 1024, 2),
         (64, 28, 128, 512, 1), (9, 14, 128, 16384, 2), (7, 28, 256, 16384, 1)]


# (mode 2: the batch-norm backward's sums, in input gradients, which have one minibatch)
@pytest.mark.parametrize("N,hw,K,OC,sets,mode", [c + (m,) for c in CASES for m in (1, 2) if (c[4], m) != (2, 2)])
def test_sums_against_64_bits(N, hw, K, OC, sets, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1804_10574_amd.ddg import load_library
    lib = load_library()
    gen = torch.Generator(device="cuda"); gen.manual_seed(5)
    M = N * hw * hw
    rows_of = lib._ZN3ddg14conv_wide_rowsEiiiiii
    rows = rows_of(M, hw, K, OC, 1, sets)
    assert 1 <= rows <= lib._ZN3ddg18conv_wide_rows_maxEi(M)
    w = (torch.randn(K * OC, device="cuda", generator=gen) * K ** -0.5).bfloat16()    # (some order of some weights: only the sums matter)
    x = [torch.randn((M, K), device="cuda", generator=gen).bfloat16() for _ in range(sets)]
    y = [torch.full((M, OC), 9.0, device="cuda", dtype=torch.bfloat16) for _ in range(sets)]
    st = [torch.full((rows + 1, 2, OC), 7.0, device="cuda") for _ in range(sets)]
    z = torch.randn((M, OC), device="cuda", generator=gen).bfloat16()
    mean, invstd = 0.1 * torch.randn(OC, device="cuda", generator=gen), 0.5 + torch.rand(OC, device="cuda", generator=gen)
    torch.cuda.synchronize()
    below = Below(2, st[0].data_ptr(), None, None, None, z.data_ptr(), mean.data_ptr(), invstd.data_ptr())
    second = Second(x[-1].data_ptr(), y[-1].data_ptr(), st[-1].data_ptr(), None, None)
    launch = lib._ZN3ddg16conv_wide_launchEPKvS1_PvPfS1_S1_iiiiiiP12ihipStream_tPKfS7_PKNS_14ConvWideSecondEPKNS_8ConvStatE
    p = C.c_void_p
    print(f"case wide statistics {N}x{hw}x{hw} {K}-{OC} sets={sets} mode={mode} rows={rows}", flush=True)
    assert launch(p(x[0].data_ptr()), p(w.data_ptr()), p(y[0].data_ptr()), p(st[0].data_ptr() if mode == 1 else None), p(None), p(None), N, hw, hw, K,
                  OC, 1, p(None), p(None), p(None), C.byref(second) if sets == 2 else None, C.byref(below) if mode == 2 else None) == 0
    torch.cuda.synchronize()
    tiles = (M + 63) // 64
    for yk, sk in zip(y, st):
        assert bool((sk[rows] == 7.0).all())             # no more rows than announced
        got = sk[:rows].double().sum(0)
        d = yk.double()
        q = d * d if mode == 1 else d * ((z.double() - mean.double()) * invstd.double())
        f = d.float() if mode == 1 else (z.float() - mean) * invstd       # (rounded as the kernels round it)
        es, eq = float((got[0] - d.sum(0)).norm()), float((got[1] - q.sum(0)).norm())
        fs, fq = float((former(yk.float()) - d.sum(0)).norm()), float((former(yk.float(), f) - q.sum(0)).norm())
        print(f"  sums {es:.2e}, with a row per 64 pixels {fs:.2e}; second sums {eq:.2e}, {fq:.2e}", flush=True)
        # Rows of one tile: the 32 sums of a tile are added exactly and rounded once, where the former order rounds the last sum as well and 31
        # before it. Sums of bf16 values are mostly exact, so which of the few roundings fall where decides: at most a rounding, 2^-24 / sqrt(3)
        # (2-norm over many), of each tile's sum, whose square is 64 squares of a value.
        if rows == tiles:
            fs = max(fs, 2.0 ** -24 * float((64 * tiles / 3 * (d * d).mean(0)).sum().sqrt()))
        assert es <= fs and eq <= fq


def test_infinite_sums_stay_infinite():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1804_10574_amd.ddg import load_library
    lib = load_library()
    N, hw, K, OC = 9, 28, 128, 16384                      # rows with rests
    M = N * hw * hw
    rows = lib._ZN3ddg14conv_wide_rowsEiiiiii(M, hw, K, OC, 1, 1)
    x = torch.zeros((M, K), device="cuda", dtype=torch.bfloat16)
    x[M // 2] = 3e38                                      # a stored value near the largest, whose square is infinite
    w = torch.zeros(K * OC, device="cuda", dtype=torch.bfloat16)
    w[::K] = 1.0
    y, st = torch.zeros((M, OC), device="cuda", dtype=torch.bfloat16), torch.zeros((rows, 2, OC), device="cuda")
    torch.cuda.synchronize()
    p = C.c_void_p
    launch = lib._ZN3ddg16conv_wide_launchEPKvS1_PvPfS1_S1_iiiiiiP12ihipStream_tPKfS7_PKNS_14ConvWideSecondEPKNS_8ConvStatE
    print("case wide statistics infinite", flush=True)
    assert launch(p(x.data_ptr()), p(w.data_ptr()), p(y.data_ptr()), p(st.data_ptr()), p(None), p(None), N, hw, hw, K, OC, 1, p(None), p(None),
                  p(None), None, None) == 0
    torch.cuda.synchronize()
    got, d = st.double().sum(0), y.double()
    big = d.abs().amax(0) > 1e30
    assert int(big.sum()) > 0
    ref = (d.float() ** 2).sum(0)
    assert bool(((got[1] == float("inf")) == (ref == float("inf"))).all()) and bool((got[1][big] == float("inf")).all())
