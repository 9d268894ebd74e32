"""The library's own launchers and kernels, called from a test without a module around them: argument structures as csrc/ddg_kernels.h lays them out."""
import ctypes as C

P = C.c_void_p
F32, BF16 = 0, 1


class ConvArgs(C.Structure):
    _fields_ = [(n, P) for n in ("in_", "wpack", "out", "stat", "in_b", "out_b", "stat_b", "add_g", "add_mask", "proj_in", "proj_wpack")] + \
               [(n, C.c_int) for n in ("N", "IH", "IW", "IC", "OH", "OW", "OC", "R", "stride", "pad", "log2cp", "ntaps", "ksteps", "M", "dgrad", "dtype",
                                       "grid_x", "mb", "nb")]


class WgradArgs(C.Structure):
    _fields_ = [(n, P) for n in ("x", "dz", "partial", "dW")] + \
               [(n, C.c_int) for n in ("N", "H", "W", "Cin", "P", "Q", "Cout", "R", "stride", "pad", "log2cp", "J", "JB", "M", "msplit", "steps", "jgroups",
                                       "dtype", "vec")]


def lib():
    from paper_1804_10574_amd.ddg import load_library
    return load_library()


def conv_args(N, H, W, cin, cout, stride, dtype, dgrad=0):
    """A planned 3x3 convolution of cin x H x W images (dgrad: its input gradient), and the elements of its packed operand."""
    a = ConvArgs()
    p, q = (H - 1) // stride + 1, (W - 1) // stride + 1
    small, large = (p, q, cout), (H, W, cin)
    (a.IH, a.IW, a.IC), (a.OH, a.OW, a.OC) = (small, large) if dgrad else (large, small)
    a.N, a.R, a.stride, a.pad, a.ntaps, a.M, a.dgrad, a.dtype = N, 3, stride, 1, 9, N * a.OH * a.OW, dgrad, dtype
    l2, ks = C.c_int(), C.c_int()
    f = lib()._ZN3ddg16conv_wpack_elemsEiiiiPiS0_
    f.restype = C.c_size_t
    n = f(a.IC, a.OC, 3, dtype, C.byref(l2), C.byref(ks))
    a.log2cp, a.ksteps = l2.value, ks.value
    lib()._ZN3ddg9conv_planERNS_8ConvArgsE(C.byref(a))
    return a, n


def pack(w, a, n):
    """Weights [cout][cin][3][3] (fp32, on the GPU) as the operand of a planned convolution."""
    import torch
    out = torch.zeros(n, device="cuda", dtype=torch.bfloat16 if a.dtype == BF16 else torch.float32)
    torch.cuda.synchronize()
    assert lib()._ZN3ddg19pack_weights_launchEPKfPviiiiiP12ihipStream_t(P(w.data_ptr()), P(out.data_ptr()), w.shape[0], w.shape[1], 3, a.dgrad, a.dtype, P(None)) == 0
    return out


def conv(a, other=None):
    assert lib()._ZN3ddg11conv_launchERKNS_8ConvArgsEP12ihipStream_tPS1_(C.byref(a), P(None), C.byref(other) if other else None) == 0


def wgrad_args(N, H, W, cin, cout, dtype):
    """A planned weight gradient of a 3x3 convolution of stride 1."""
    a = WgradArgs()
    a.N, a.H, a.W, a.Cin, a.P, a.Q, a.Cout, a.R, a.stride, a.pad, a.M, a.dtype = N, H, W, cin, H, W, cout, 3, 1, 1, N * H * W, dtype
    lib()._ZN3ddg10wgrad_planERNS_9WgradArgsE(C.byref(a))
    return a


def wgrad(a):
    assert lib()._ZN3ddg12wgrad_launchERKNS_9WgradArgsEP12ihipStream_t(C.byref(a), P(None)) == 0


class Dim3(C.Structure):
    _fields_ = [(n, C.c_uint) for n in "xyz"]


def launch(kernel, grid, threads, *args):
    """One of the library's kernels, by its handle's name, on the default stream."""
    run = lib().hipLaunchKernel
    run.argtypes = [P, Dim3, Dim3, C.POINTER(P), C.c_size_t, P]
    ptrs = (P * len(args))(*[C.cast(C.pointer(a), P) for a in args])
    assert run(C.addressof(C.c_char.in_dll(lib(), kernel)), Dim3(*grid), Dim3(threads, 1, 1), ptrs, 0, None) == 0
