"""Weight gradients of wide layers, several of which share a launch: modules whose layers close a launch by their number,
by the places on the chip inside a block, with slices cut because a sum would get too long and because places
are left, and with tap shifts on images narrower than a step; against the oracle, the parameters of every block apart."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu

CASES = [(9, 2, 3, 128, 128),      # 27 layers: more than a launch takes
         (8, 1, 5, 1024, 256),     # 25 pixels, one step: 544 tiles for 512 places
         (1, 50, 8, 128, 128),     # 3200 pixels, 50 steps: one more than a slice may have
         (2, 130, 7, 256, 128),    # 6370 pixels, ragged last step, several image rows per advance
         (1, 129, 8, 512, 128)]    # 129 statistics rows behind the 512-channel layers, 43 behind the 128-channel 1x1 layer


@pytest.mark.parametrize("blocks,batch,hw,c,cmid", CASES)
def test_weight_gradients_of_many_wide_layers(blocks, batch, hw, c, cmid):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from paper_1804_10574_amd.ddg import make_desc
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    print(f"case {blocks} wide blocks batch={batch} hw={hw} {c}-{cmid}-{c}", flush=True)
    net, shape = [(wk.BLOCK_BOTTLENECK, c, cmid, c, 1, 0)] * blocks, (batch, c, hw, hw)
    mod = ddg.Module(make_desc(2, 2, batch, (c, hw, hw), net, 0, ddg.DDG_BF16, 0.9, 0.0, 1e-5))
    oracle = orc.OracleNet(2, [net], batch, (c, hw, hw), 0, 0.9, 0.0, 1e-5, "f64", k_first=2, store_bf16=True)
    n = oracle.param_count(2)
    theta = (wk.normal(31, 1, n) * 0.05 + 0.02).astype(np.float32)
    oracle.set_params(2, theta.astype(np.float64))
    mod.set_params(theta)

    class WL:
        dtype = "bf16"
    h_in = wk.normal(33, 0, int(np.prod(shape))).reshape(shape)
    delta = wk.normal(37, 0, int(np.prod(shape))).reshape(shape)
    hd, dd = H.to_dev_nhwc(h_in, WL), H.to_dev_nhwc(delta, WL)
    h_out, d_out = torch.empty_like(hd), torch.zeros_like(hd)
    torch.cuda.synchronize()
    mod.forward(0, hd, h_out)
    mod.backward_delayed(0, delta_in=dd, delta_out=d_out)
    mod.sync()
    oracle.forward(2, 0, H.from_dev_nhwc(hd))
    oracle.backward_delayed(2, 0, H.from_dev_nhwc(dd), None, in_shape=shape)
    got, ref = mod.get_grad().reshape(blocks, -1), oracle.get_grad(2).reshape(blocks, -1)
    errs = [H.rel_err(got[b], ref[b]) for b in range(blocks)]
    print("  " + " ".join(f"{e:.1e}" for e in errs), flush=True)
    # the two sides round at the same points; a sum that falls on the other side of a rounding boundary flips a ReLU decision
    # near zero: a fraction f < 1e-3 per ReLU, of which 3 lie in a block: sqrt(3 f blocks above)
    for b, e in enumerate(errs):
        assert e <= (3e-3 * (blocks - b)) ** 0.5
    mod.close()
