"""Layers with more than 64 channels at the sizes where their kernels can go wrong, one bottleneck block
as module 2 of 3 (delay 1) against the oracle: pixel counts below one tile, ragged, exactly at
and just above the line up to which the elementwise kernels finalise the statistics, rows that wrap inside
a tile, one channel group and several, a projection (two sets of statistics meet in one kernel)."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu

# (dtype, batch, height = width, cin, cmid, cout, projection): what the size is there for
CASES = [("bf16", 1, 5, 128, 128, 128, 0),       # 25 pixels: less than one tile
         ("bf16", 3, 15, 512, 128, 512, 0),      # 675 pixels: ragged tiles that span image rows and images
         ("bf16", 8, 32, 128, 128, 128, 0),      # 8192 pixels = 128 statistics rows: the last size finalised by the consumers (64-pixel rows)
         ("bf16", 129, 8, 128, 128, 128, 0),     # 8256 pixels = 129 rows: finalise launches (64-pixel rows; the 3x3 layer writes 65)
         ("bf16", 16, 32, 128, 128, 128, 0),     # 16384 pixels = 128 rows of the 3x3 layer's 128 pixels: the last size
         ("bf16", 257, 8, 128, 128, 128, 0),     # 16448 pixels = 129 of them
         ("bf16", 2, 12, 256, 256, 512, 1),      # projection, several channel groups everywhere
         ("bf16", 2, 40, 128, 256, 128, 0),      # rows longer than a tile's halo of a 14 x 14 image
         ("bf16", 1, 31, 128, 512, 128, 0),      # the widest image whose halo fits, four slices
         ("bf16", 7, 1, 128, 128, 128, 0),       # 1 x 1 images: no neighbour exists
         ("f32", 3, 9, 128, 128, 256, 1)]


@pytest.mark.parametrize("dtype,batch,hw,cin,cmid,cout,proj", CASES)
def test_one_wide_block_matches_the_oracle(dtype, batch, hw, cin, cmid, cout, proj):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    print(f"case wide block {dtype} batch={batch} hw={hw} {cin}-{cmid}-{cout} proj={proj}", flush=True)
    blocks = [(wk.BLOCK_BOTTLENECK, cin, cmid, cout, 1, proj)]
    shape = (batch, cin, hw, hw)
    mod = ddg.Module(make_desc(3, 2, batch, (cin, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32,
                               0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(3, [blocks], batch, (cin, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=2,
                           store_bf16=(dtype == "bf16"))
    n = oracle.param_count(2)
    theta = (wk.normal(11, 1, n) * 0.05 + 0.02).astype(np.float32)
    oracle.set_params(2, theta.astype(np.float64))
    mod.set_params(theta)

    class WL:
        pass
    wl = WL(); wl.dtype = dtype
    # fp32: sums of up to 2304 products and 8256 pixels in another order. bf16: the two sides round at
    # the same points; where a sum falls on the other side of a rounding boundary a value differs by 2^-9
    # and a ReLU decision near zero flips (two ReLU layers between the error gradient and dx: a
    # fraction f of flipped decisions moves the gradient by about sqrt(f), f < 1e-3 here)
    tol_h, tol_g = (1e-4, 1e-3) if dtype == "f32" else (2e-2, 4e-2)
    for t in range(3):
        h_in = wk.normal(13, t, int(np.prod(shape))).reshape(shape)
        delta = wk.normal(17, t, batch * cout * hw * hw).reshape(batch, cout, hw, hw)
        hd, dd = H.to_dev_nhwc(h_in, wl), H.to_dev_nhwc(delta, wl)
        if dtype == "bf16":
            h_in, delta = H.from_dev_nhwc(hd), H.from_dev_nhwc(dd)
        h_out = torch.empty((batch, hw, hw, cout), dtype=H.tdtype(wl), device="cuda")
        d_out = torch.zeros_like(hd)
        torch.cuda.synchronize()
        mod.forward(t, hd, h_out)
        did = mod.backward_delayed(t, delta_in=dd, delta_out=d_out)
        mod.sync()
        ref_h = oracle.forward(2, t, h_in)
        ref_did, ref_dout, _ = oracle.backward_delayed(2, t, delta, None, in_shape=shape)
        assert did == bool(ref_did) == (t >= 1)
        e_h = H.rel_err(H.from_dev_nhwc(h_out), ref_h)
        print(f"  t={t} h {e_h:.2e}", flush=True)
        assert e_h <= tol_h
        if did:
            e_d, e_g = H.rel_err(H.from_dev_nhwc(d_out), ref_dout), H.rel_err(mod.get_grad(), oracle.get_grad(2))
            print(f"  t={t} dx {e_d:.2e} grad {e_g:.2e}", flush=True)
            assert e_d <= tol_g and e_g <= tol_g
        mod.update(t, 0.0)
        oracle.update(2, 0.0)
    mod.close()


@pytest.mark.parametrize("mode", ["stale_jacobian", "forward_stream"])
@pytest.mark.parametrize("dtype,batch,hw,cin,cmid,cout,proj", [("bf16", 3, 15, 512, 128, 512, 0), ("bf16", 2, 12, 256, 256, 512, 1),
                                                               ("f32", 3, 9, 128, 128, 256, 1)])
def test_two_wide_blocks_in_the_other_modes(mode, dtype, batch, hw, cin, cmid, cout, proj):
    """Statistics finalised by the elementwise kernels, for every kept tape of stale-Jacobian mode and for the forward
    pass on a stream of its own (unpaired passes), as module 2 of 4 (delay 2) with weights that move."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    print(f"case wide blocks {mode} {dtype} batch={batch} hw={hw} {cin}-{cmid}-{cout} proj={proj}", flush=True)
    blocks = [(wk.BLOCK_BOTTLENECK, cin, cmid, cout, 1, proj), (wk.BLOCK_BOTTLENECK, cout, cmid, cout, 1, 0)]
    shape, stale = (batch, cin, hw, hw), mode == "stale_jacobian"
    streams = [torch.cuda.Stream() for _ in range(2)]
    mod = ddg.Module(make_desc(4, 2, batch, (cin, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32,
                               0.9, 0.0, 1e-5, stream=streams[0].cuda_stream, stale_jacobian=stale,
                               forward_stream=None if stale else streams[1].cuda_stream))
    oracle = orc.OracleNet(4, [blocks], batch, (cin, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=2, stale_jacobian=stale,
                           store_bf16=(dtype == "bf16"))
    theta = (wk.normal(11, 3, oracle.param_count(2)) * 0.05 + 0.02).astype(np.float32)
    oracle.set_params(2, theta.astype(np.float64))
    mod.set_params(theta)

    class WL:
        pass
    wl = WL(); wl.dtype = dtype
    # as above, but four ReLU layers between the error gradient and dx instead of two: independent flips of a fraction
    # f < 1e-3 in each add up to sqrt(4 f) = 6.3e-2
    tol_h, tol_g = (1e-4, 1e-3) if dtype == "f32" else (2e-2, 6e-2)
    hs = []                                                            # (inputs stay alive until the streams are done)
    for t in range(5):
        h_in = wk.normal(13, 20 + t, int(np.prod(shape))).reshape(shape)
        delta = wk.normal(17, 20 + t, batch * cout * hw * hw).reshape(batch, cout, hw, hw)
        hd, dd = H.to_dev_nhwc(h_in, wl), H.to_dev_nhwc(delta, wl)
        if dtype == "bf16":
            h_in, delta = H.from_dev_nhwc(hd), H.from_dev_nhwc(dd)
        h_out = torch.empty((batch, hw, hw, cout), dtype=H.tdtype(wl), device="cuda")
        d_out = torch.zeros_like(hd)
        hs += [hd, dd, h_out, d_out]
        torch.cuda.synchronize()
        mod.forward(t, hd, h_out)
        did = mod.backward_delayed(t, delta_in=dd, delta_out=d_out)
        mod.sync()
        ref_h = oracle.forward(2, t, h_in)
        ref_did, ref_dout, _ = oracle.backward_delayed(2, t, delta, None, in_shape=shape)
        assert did == bool(ref_did) == (t >= 2)
        e_h = H.rel_err(H.from_dev_nhwc(h_out), ref_h)
        print(f"  t={t} h {e_h:.2e}", flush=True)
        assert e_h <= tol_h
        if did:
            e_d, e_g = H.rel_err(H.from_dev_nhwc(d_out), ref_dout), H.rel_err(mod.get_grad(), oracle.get_grad(2))
            print(f"  t={t} dx {e_d:.2e} grad {e_g:.2e}", flush=True)
            assert e_d <= tol_g and e_g <= tol_g
        mod.update(t, 1e-5)
        oracle.update(2, 1e-5)
    mod.close()


# the stride-2 input gradient by pixel parity: odd and even heights, one pixel, a single row of tiles, all widths that
# select one, two and four k-steps per tap, with a projection (its own stride-2 1x1 launch and the sum of the two)
# (1 x 1 images in a batch of 5: with a single pixel per channel the batch norm's gradient is exactly zero, and a relative
# error against rounding noise says nothing)
S2_CASES = [("f32", 2, 9, 16, 32), ("f32", 5, 1, 32, 64), ("f32", 65, 32, 16, 32), ("f32", 3, 7, 32, 64),
            ("bf16", 2, 9, 16, 32), ("bf16", 3, 2, 32, 64), ("bf16", 130, 32, 16, 32), ("bf16", 2, 11, 64, 128),
            ("bf16", 5, 16, 32, 64)]


@pytest.mark.parametrize("dtype,batch,hw,cin,cout", S2_CASES)
def test_stride_two_block_matches_the_oracle(dtype, batch, hw, cin, cout):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    print(f"case stride-two block {dtype} batch={batch} hw={hw} {cin}-{cout}", flush=True)
    blocks = [(wk.BLOCK_BASIC, cin, 0, cout, 2, 1)]
    shape, ho = (batch, cin, hw, hw), (hw - 1) // 2 + 1
    mod = ddg.Module(make_desc(2, 2, batch, (cin, hw, hw), blocks, 0, ddg.DDG_BF16 if dtype == "bf16" else ddg.DDG_F32,
                               0.9, 0.0, 1e-3))
    oracle = orc.OracleNet(2, [blocks], batch, (cin, hw, hw), 0, 0.9, 0.0, 1e-3, "f64", k_first=2,
                           store_bf16=(dtype == "bf16"))
    theta = (wk.normal(21, 1, oracle.param_count(2)) * 0.1 + 0.05).astype(np.float32)
    oracle.set_params(2, theta.astype(np.float64))
    mod.set_params(theta)

    class WL:
        pass
    wl = WL(); wl.dtype = dtype
    h_in = wk.normal(23, 0, int(np.prod(shape))).reshape(shape)
    delta = wk.normal(27, 0, batch * cout * ho * ho).reshape(batch, cout, ho, ho)
    hd, dd = H.to_dev_nhwc(h_in, wl), H.to_dev_nhwc(delta, wl)
    if dtype == "bf16":
        h_in, delta = H.from_dev_nhwc(hd), H.from_dev_nhwc(dd)
    h_out = torch.empty((batch, ho, ho, cout), dtype=H.tdtype(wl), device="cuda")
    d_out = torch.full_like(hd, float("nan"))
    torch.cuda.synchronize()
    mod.forward(0, hd, h_out)
    mod.backward_delayed(0, delta_in=dd, delta_out=d_out)
    mod.sync()
    ref_h = oracle.forward(2, 0, h_in)
    _, ref_d, _ = oracle.backward_delayed(2, 0, delta, None, in_shape=shape)
    e_h, e_d = H.rel_err(H.from_dev_nhwc(h_out), ref_h), H.rel_err(H.from_dev_nhwc(d_out), ref_d)
    print(f"  h {e_h:.2e} dx {e_d:.2e}", flush=True)
    # as above; one ReLU layer lies between the error gradient and dx
    assert e_h <= (1e-4 if dtype == "f32" else 2e-2) and e_d <= (1e-3 if dtype == "f32" else 3e-2)
    mod.close()
