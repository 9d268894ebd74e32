"""The evaluation kernel that keeps activations in LDS across layers, against the oracle: both
operand types (bf16: whole images, or strips of rows; fp32: strips), pixel counts that fill no 16-pixel block,
odd heights under stride 2, one and several images, one large image (strips in bf16 too), a
module whose stages together exceed LDS, a module that starts with a block between stages, and every channel
count as first and last. The launches that ran are counted, and no other convolution kernel may have."""
import numpy as np
import pytest

import workloads as wk
from tests.eval_plan import launches, shapes
from workloads.configs import custom_cifar

pytestmark = pytest.mark.gpu

# (units, cuts, batch, image size): what the size is there for. bf16: the modules are one launch each but where it says strips
CASES = [(1, [2, 3], 1, 32),        # one image; modules that start with a block between stages
         (1, [], 3, 10),            # 100 / 25 / 9 pixels: ragged everywhere, odd sizes under stride 2
         (2, [3, 5], 2, 24),        # 576 / 144 / 36 pixels
         (3, [4, 7], 2, 28),        # runs of identity blocks at 16, 32 and 64 channels
         (1, [1, 2], 1, 44),        # one large image: strips of a row or two
         (1, [], 2, 32),            # a whole network
         (2, [], 2, 40), (1, [], 20, 56)]   # networks whose buffers exceed LDS: strips of a row or two, and of several
STRIPS = {(1, 1, 44), (2, 2, 40), (1, 20, 56)}     # (units, batch, image size)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("units,cuts,batch,hw", CASES)
def test_fused_evaluation_matches_the_oracle(dtype, units, cuts, batch, hw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from oracle import ddg_oracle as orc
    from tests import gpu_harness as H
    wl = custom_cifar(units, cuts, batch=batch, num_classes=7, hw=hw, dtype=dtype, name="eval_fused")
    K = wl.K
    print(f"case fused evaluation {dtype} units={units} cuts={cuts} batch={batch} hw={hw}", flush=True)
    pipe = ddg.Pipeline(H.descs_for(wl), [torch.cuda.Stream().cuda_stream for _ in range(K)])
    mods = {k: pipe.module(k) for k in range(1, K + 1)}
    oracle = orc.OracleNet.from_workload(wl, dtype="f64")
    H.init_both(wl, mods, oracle)
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    logits = torch.zeros((batch, wl.num_classes), dtype=torch.float32, device="cuda")
    # two iterations with step size 0 move the running estimates away from 0 and 1
    for t in range(2):
        x, y = wk.minibatch(wl, t)
        xd, yd = H.to_dev_nhwc(x, wl), torch.from_numpy(y).to("cuda")
        torch.cuda.synchronize()
        pipe.step(xd, yd, 0.0, loss)
        oracle.ddg_step(H.from_dev_nhwc(xd) if dtype == "bf16" else x, y, 0.0)
    pipe.sync()
    x, y = wk.minibatch(wl, 9)
    xd, yd = H.to_dev_nhwc(x, wl), torch.from_numpy(y).to("cuda")
    torch.cuda.synchronize()
    for m in mods.values():
        m.profile_enable(True)
    pipe.forward_eval(xd, yd, loss, logits)
    for m in wl.modules:
        ran = {kind: v[0] for kind, v in mods[m.k].profile_read().items() if v[0]}
        body = shapes([b.as_tuple() for b in m.blocks])
        plan = launches(body, batch, m.in_h, dtype == "bf16") if body else []
        assert ran == ({"eval_blocks": len(plan)} if body else {}), (m.k, ran)
        if dtype == "bf16":
            if (units, batch, hw) in STRIPS:
                assert len(plan) == len(body) and all(l[1] > 1 for l in plan)
            else:
                assert len(plan) <= 1
    h = H.from_dev_nhwc(xd) if dtype == "bf16" else x
    for k in range(1, K):
        h = oracle.forward_eval(k, h)
    ref_loss, ref_logits = oracle.forward_eval(K, h, y)
    # fp32: sums of up to 576 products in another order; bf16: the two sides round at the same points and
    # differ where a sum falls on the other side of a rounding boundary (2^-9 of one value)
    tol = 1e-4 if dtype == "f32" else 2e-2
    e = H.rel_err(logits.cpu().numpy(), ref_logits)
    print(f"  logits {e:.2e}", flush=True)
    assert e <= tol
    assert abs(float(loss.cpu()[0]) - ref_loss) <= tol * abs(ref_loss)
    pipe.close()
