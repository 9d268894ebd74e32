"""The convolutions that derive their on-load batch norm from the producer's statistics rows, called through the library's own launchers,
against the same launch with scale and shift given: rows around what a thread holds at once, of one and two minibatches. What lies behind the
rows in memory is no part of the sums."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


class Second(C.Structure):     # ConvWideSecond
    _fields_ = [(n, C.c_void_p) for n in ("in_", "out", "stat", "scale", "shift")]


class Rows(C.Structure):       # BnRows
    _fields_ = [("partial", C.c_void_p), ("rows", C.c_int), ("gamma", C.c_void_p), ("beta", C.c_void_p), ("inv_count", C.c_double),
                ("eps", C.c_float)] + [(n, C.c_void_p) for n in ("mean", "invstd", "scale", "shift")]


# 512 threads share rows of K channels: 1024/K rows at a time, 14 times
@pytest.mark.parametrize("K,R,rows", [(128, 1, 1), (128, 1, 112), (128, 1, 113), (128, 1, 256), (256, 1, 3), (256, 1, 56), (256, 1, 57), (256, 1, 128),
                                      (128, 3, 5), (256, 3, 55), (256, 3, 98), (256, 3, 128), (128, 3, 256)])
@pytest.mark.parametrize("sets", [1, 2])
def test_from_rows(K, R, rows, sets):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1804_10574_amd.ddg import load_library
    lib = load_library()
    N, hw, OC = 3, 7, 256
    M = N * hw * hw
    assert lib._ZN3ddg20conv_wide_takes_rowsEiiii(K, hw, R, rows) & 0xff == 1
    assert lib._ZN3ddg20conv_wide_takes_rowsEiiii(K, hw, R, 32768 // K + 1) & 0xff == 0
    assert lib._ZN3ddg20conv_wide_takes_rowsEiiii(512, hw, 3, 1) & 0xff == 0          # (keeps its finalise launch)
    gen = torch.Generator(device="cuda"); gen.manual_seed(K + rows)
    f = dict(device="cuda", generator=gen)
    w = (torch.randn(R * R * K * OC, **f) * (R * R * K) ** -0.5).bfloat16()     # (some order of some weights)
    x = [torch.randn((M, K), **f).bfloat16() for _ in range(sets)]
    gamma, beta, eps, count = 1 + 0.2 * torch.randn(K, **f), 0.3 * torch.randn(K, **f), 1e-5, 64.0 * rows
    part = []
    for _ in range(sets):
        v = torch.randn((rows, 64, K), **f) * 1.5 + 0.4
        # in memory behind the rows: as many as a workgroup requests at once, twice
        part.append(torch.cat([torch.stack([v.sum(1), (v * v).sum(1)], 1), torch.full((2 * 14 * 1024 // K, 2, K), float("nan"), device="cuda")]))
    stats = lib._ZN3ddg14conv_wide_rowsEiiiiii
    nst = stats(M, hw, K, OC, R, sets)
    vec = [torch.full((4, K), 9.0, device="cuda") for _ in range(sets)]        # mean, invstd, scale, shift
    exact = []
    for p in part:
        s = p[:rows].double().sum(0)
        mu = s[0] / count
        inv = ((s[1] / count - mu * mu).clamp_min(0) + eps).rsqrt()
        sc = gamma * inv.float()
        exact.append(torch.stack([mu.float(), inv.float(), sc, beta - mu.float() * sc]).contiguous())

    def out():
        return [torch.full((M, OC), 7.0, device="cuda", dtype=torch.bfloat16) for _ in range(sets)], [torch.zeros((nst, 2, OC), device="cuda") for _ in range(sets)]
    (y0, s0), (y1, s1) = out(), out()
    torch.cuda.synchronize()
    P = C.c_void_p
    ptr = lambda t: P(t.data_ptr())
    given = lib._ZN3ddg16conv_wide_launchEPKvS1_PvPfS1_S1_iiiiiiP12ihipStream_tPKfS7_PKNS_14ConvWideSecondEPKNS_8ConvStatE
    derived = lib._ZN3ddg21conv_wide_rows_launchEPKvS1_PvPfiiiiiiP12ihipStream_tPKNS_6BnRowsEPKNS_14ConvWideSecondE
    second = Second(x[-1].data_ptr(), y0[-1].data_ptr(), s0[-1].data_ptr(), exact[-1][2].data_ptr(), exact[-1][3].data_ptr())
    r = given(ptr(x[0]), ptr(w), ptr(y0[0]), ptr(s0[0]), None, None, N, hw, hw, K, OC, R, None, ptr(exact[0][2]), ptr(exact[0][3]),
              C.byref(second) if sets == 2 else None, None)
    assert r == 0
    arr = (Rows * 2)(*[Rows(part[i % sets].data_ptr(), rows, gamma.data_ptr(), beta.data_ptr(), 1.0 / count, eps, *[vec[i % sets][j].data_ptr() for j in range(4)])
                       for i in range(2)])
    second = Second(x[-1].data_ptr(), y1[-1].data_ptr(), s1[-1].data_ptr(), None, None)
    r = derived(ptr(x[0]), ptr(w), ptr(y1[0]), ptr(s1[0]), N, hw, hw, K, OC, R, None, arr, C.byref(second) if sets == 2 else None)
    assert r == 0
    torch.cuda.synchronize()
    for i in range(sets):
        # the sums are fp64 in another order: a value may round to the next fp32 number, scale and shift after two more roundings
        assert torch.allclose(vec[i], exact[i], rtol=4e-7, atol=4e-7)
        # an activation may then round to its bf16 neighbour (2^-8 of it), few do; a sum of R*R*K products moves by far less than a value's scale
        a, b = y0[i].float(), y1[i].float()
        assert (a - b).abs().max() <= 2.0 ** -6 * a.abs().max()
        assert ((a != b).float().mean()) < 0.05
        t0, t1 = s0[i].double().sum(0), s1[i].double().sum(0)
        assert (t0 - t1).abs().max() <= 1e-3 * M ** 0.5 * a.abs().max() ** 2
