"""First layers of a network (few input channels, pixels staged in LDS): every channel count and tile shape they take, images of one pixel, one row
and one column, rows as wide as the staging allows and one wider (the generic kernels), against the oracle; the same, and the edges of the staging's
other limits, against the generic kernels bit for bit; and small tiles of the generic kernels."""
import ctypes as C

import numpy as np
import pytest

import workloads as wk
from tests import launchers as L
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu
H = parity.H

# input channels, output channels, images, height, width
STEMS = {"one_pixel": (3, 16, 64, 1, 1), "one_row": (3, 16, 8, 1, 9), "one_column": (3, 16, 8, 9, 1), "ragged": (3, 16, 2, 5, 7), "one_tile": (3, 16, 4, 8, 8), "one_channel": (1, 16, 2, 6, 9), "c32": (2, 32, 2, 9, 4),
         "c64_four_channels": (4, 64, 2, 7, 11), "c32_tiles": (3, 32, 9, 30, 31), "c64_tiles": (3, 64, 5, 31, 30), "c32_all_blocks": (3, 32, 17, 31, 32), "c64_all_blocks": (3, 64, 17, 31, 32),
         "widest": (3, 16, 3, 5, 127), "wider": (3, 16, 3, 5, 128), "many_trips": (3, 16, 130, 32, 32), "tall_many_channels": (5, 16, 2, 9, 8)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(STEMS))
def test_first_layer(H, which, dtype):
    import torch
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    cin, cout, N, h, w = STEMS[which]
    print(f"case first layer {which} {dtype}", flush=True)
    blocks = [(wk.BLOCK_STEM, cin, 0, cout, 1, 0)]
    mod = ddg.Module(make_desc(2, 1, N, (cin, h, w), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(2, [blocks], N, (cin, h, w), 0, 0.9, 0.0, 1e-5, "f64", k_first=1, store_bf16=(dtype == "bf16"))
    theta = (wk.normal(11, 1, mod.param_count()) * 0.2 + 0.05).astype(np.float32)
    mod.set_params(theta)
    oracle.set_params(1, theta.astype(np.float64))

    class WL:
        pass
    wl = WL(); wl.dtype = dtype
    for t in range(3):          # (from t = 1 on two minibatches a launch)
        x = wk.normal(13, t, N * cin * h * w).reshape(N, cin, h, w)
        d = wk.normal(17, t, N * cout * h * w).reshape(N, cout, h, w)
        xd, dd = H.to_dev_nhwc(x, wl), H.to_dev_nhwc(d, wl)
        x, d = H.from_dev_nhwc(xd), H.from_dev_nhwc(dd)
        out = torch.empty((N, h, w, cout), dtype=H.tdtype(wl), device="cuda")
        torch.cuda.synchronize()
        mod.forward(t, xd, out)
        did = mod.backward_delayed(t, delta_in=dd)
        mod.sync()
        ref = oracle.forward(1, t, x)
        ref_did, _, _ = oracle.backward_delayed(1, t, d, None, in_shape=x.shape)
        assert did == bool(ref_did) == (t >= 1)
        tol = parity.TOL[dtype]
        e = H.rel_err(H.from_dev_nhwc(out), ref)
        assert e < tol, (t, e)
        if did:
            e = H.rel_err(mod.get_grad(), oracle.get_grad(1))
            assert e < tol, (t, e)
        mod.update(t, 0.0)
        oracle.update(1, 0.0)
    mod.close()


def _rand(shape, dtype, seed):
    import torch
    gen = torch.Generator(device="cuda"); gen.manual_seed(seed)
    x = torch.randn(shape, device="cuda", generator=gen)
    return x.bfloat16() if dtype == L.BF16 else x


# and as many pixels as have their places from fp32 divisions (below 2^22), of one image and of many, and a row more
CONVS = dict(STEMS, below_2_22=(3, 16, 1, 33026, 127), images_below_2_22=(3, 16, 466, 100, 90), above_2_22=(3, 16, 1, 33027, 127), two_images_2_22=(3, 16, 2, 32769, 67))


@pytest.mark.parametrize("dtype", [L.F32, L.BF16])
@pytest.mark.parametrize("sets", [1, 2])
@pytest.mark.parametrize("which", sorted(CONVS))
def test_forward_has_the_bits_of_the_generic_kernel(which, sets, dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cin, cout, N, h, w = CONVS[which]
    print(f"case stem forward {which} sets {sets} dtype {dtype}", flush=True)
    a, n = L.conv_args(N, h, w, cin, cout, 1, dtype)
    staged = bool(L.lib()._ZN3ddg12stem_conv_okERKNS_8ConvArgsE(C.byref(a)) & 0xff)
    assert staged == (cin <= (4 if dtype == L.BF16 else 3) and 64 * a.mb + 2 * w + 2 <= 512)
    wp = L.pack(_rand((cout, cin, 3, 3), L.F32, 1) * 0.3, a, n)
    x = [_rand((N, h, w, cin), dtype, 2 + i) for i in range(sets)]
    results = []
    for generic in (False, True):
        out = [torch.full((a.M, cout), 7.0, device="cuda", dtype=x[0].dtype) for _ in range(2 * sets)]
        stat = [torch.full((a.grid_x, 2, cout), 9.0, device="cuda") for _ in range(2 * sets)]
        ab = []
        for c in range(2):           # (only the generic kernel takes two convolutions: the same one twice)
            b = L.ConvArgs.from_buffer_copy(a)
            b.in_, b.wpack, b.out, b.stat = x[0].data_ptr(), wp.data_ptr(), out[c].data_ptr(), stat[c].data_ptr()
            if sets == 2:
                b.in_b, b.out_b, b.stat_b = x[1].data_ptr(), out[2 + c].data_ptr(), stat[2 + c].data_ptr()
            ab.append(b)
        torch.cuda.synchronize()
        L.conv(ab[0], ab[1] if generic else None)
        torch.cuda.synchronize()
        results.append([t for i in range(sets) for t in (out[2 * i], stat[2 * i])])
    for s, g in zip(*results):
        assert torch.equal(s, g)


# and as many pixels as a workgroup's share of LDS holds, and more (the generic kernel); none of them a whole number of steps
WGRADS = dict({k: v for k, v in STEMS.items() if v[0] == 3}, most_pixels=(3, 64, 374, 32, 32), more_pixels=(3, 64, 375, 32, 32), most_pixels_c16=(3, 16, 1497, 33, 31), more_pixels_c16=(3, 16, 1501, 33, 31))


@pytest.mark.parametrize("dtype", [L.F32, L.BF16])
@pytest.mark.parametrize("which", sorted(WGRADS))
def test_weight_gradient_has_the_bits_of_the_generic_kernel(which, dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cin, cout, N, h, w = WGRADS[which]
    print(f"case stem weight gradient {which} dtype {dtype}", flush=True)
    a = L.wgrad_args(N, h, w, cin, cout, dtype)
    staged = bool(L.lib()._ZN3ddg13stem_wgrad_okERKNS_9WgradArgsE(C.byref(a)) & 0xff)
    assert staged == ((16 * a.steps + 2 * w + 3) * 16 <= 48 * 1024) == (not which.startswith("more")), a.steps
    x, dz = _rand((N, h, w, cin), dtype, 5), _rand((N, h, w, cout), dtype, 6)
    results = []
    for generic in (False, True):
        part = torch.full((a.msplit, cout, a.JB * 16), 9.0, device="cuda")
        b = L.WgradArgs.from_buffer_copy(a)
        b.x, b.dz, b.partial = x.data_ptr(), dz.data_ptr(), part.data_ptr()
        torch.cuda.synchronize()
        if generic:
            L.launch("_ZN3ddg17wgrad_mfma_kernelI" + ("fLi3E" if dtype == L.F32 else "NS_6bf16_tELi3E") + "EEvNS_9WgradArgsE", (a.msplit, cout // 16, a.jgroups), 256, b)
        else:
            L.wgrad(b)
        torch.cuda.synchronize()
        results.append(part.view(a.msplit, cout, a.JB * 4, 4)[:, :, :9, :cin])      # (what the sum over the rows reads)
    assert torch.equal(*results)
    # and the sum is the gradient (fp32 products of what both read, fp64 sums of the partial tiles)
    got = results[0].double().sum(0)
    ref = torch.nn.grad.conv2d_weight(x.permute(0, 3, 1, 2).double().cpu(), (cout, cin, 3, 3), dz.permute(0, 3, 1, 2).double().cpu(), padding=1) if a.M < 200000 else None
    if ref is not None:
        ref = ref.permute(0, 2, 3, 1).reshape(cout, 9, cin)
        assert ((got.cpu() - ref).norm() / ref.norm()) < 1e-5


SMALL = {"small_c16_5": ([(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)], 1, 5), "small_c16_24": ([(wk.BLOCK_BASIC, 16, 0, 16, 1, 0)], 3, 24),
         "small_c32_7": ([(wk.BLOCK_BASIC, 32, 0, 32, 1, 0)], 5, 7), "small_c64_7": ([(wk.BLOCK_BASIC, 64, 0, 64, 1, 0)], 3, 7),
         "small_c32_to_64": ([(wk.BLOCK_BASIC, 32, 0, 64, 2, 1)], 5, 15), "small_c16_to_32": ([(wk.BLOCK_BASIC, 16, 0, 32, 2, 1)], 21, 28),
         "small_c128_6": ([(wk.BLOCK_BASIC, 128, 0, 128, 1, 0)], 2, 6)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(SMALL))
def test_small_launches(H, which, dtype, monkeypatch):
    monkeypatch.setitem(parity.SINGLE_BLOCKS, which, SMALL[which])
    parity.test_single_block_module(H, which, dtype)
