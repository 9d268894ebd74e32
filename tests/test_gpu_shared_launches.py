"""Launches that carry work of several layers: a stage's first block (3x3 and 1x1 layer forward, three weight gradients, two input
gradients) on even and ragged sizes, as the module's only block, against the oracle; and the pipeline's sums-update-repack
launch, bit for bit against the same modules driven call by call."""
import numpy as np
import pytest

import workloads as wk
from workloads.configs import custom_cifar
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu
H = parity.H

# 16 -> 32 on 31 and 32 wide images, 32 -> 64 on 15 and 16: the sizes whose second layer has 16- and 8-wide tiles; one image, several,
# and more row strips than workgroups
DOWN = {"down_c32_31": ([(wk.BLOCK_BASIC, 16, 0, 32, 2, 1)], 3, 31), "down_c32_one": ([(wk.BLOCK_BASIC, 16, 0, 32, 2, 1)], 1, 32),
        "down_c32_many": ([(wk.BLOCK_BASIC, 16, 0, 32, 2, 1)], 70, 32), "down_c64_15": ([(wk.BLOCK_BASIC, 32, 0, 64, 2, 1)], 5, 15),
        "down_c64_one": ([(wk.BLOCK_BASIC, 32, 0, 64, 2, 1)], 1, 16), "down_c64_many": ([(wk.BLOCK_BASIC, 32, 0, 64, 2, 1)], 130, 16)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(DOWN))
def test_first_block_of_a_stage(H, which, dtype, monkeypatch):
    monkeypatch.setitem(parity.SINGLE_BLOCKS, which, DOWN[which])
    parity.test_single_block_module(H, which, dtype)


# cuts inside and between stages; images whose stages are not the tiled sizes (generic layers); a classifier of 37 and of 300; a
# module that is the classifier alone
CASES = {"tiled": lambda d: custom_cifar(2, [2, 5], batch=5, num_classes=37, hw=32, dtype=d, name="tiled"),
         "generic": lambda d: custom_cifar(1, [1, 3], batch=3, num_classes=300, hw=10, dtype=d, name="generic"),
         "head_alone": lambda d: wk.resnet8((1, 3, 5, 7), batch=9, dtype=d, weight_decay=5e-4)}


@pytest.mark.parametrize("opt", ["sgd", "adam"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", sorted(CASES))
def test_pipeline_update_is_the_call_by_call_update(H, which, dtype, opt):
    import torch
    import paper_1804_10574_amd as ddg
    wl = CASES[which](dtype)
    K, steps, lr = wl.K, 2 * wl.K + 3, 0.05 if opt == "sgd" else 1e-3
    print(f"case pipeline update {which} {dtype} {opt}", flush=True)
    data = []
    for t in range(steps):
        x, y = wk.minibatch(wl, t)
        data.append((H.to_dev_nhwc(x, wl), torch.from_numpy(y).to("cuda")))
    theta = {m.k: wk.init_module_params(wl, m, perturb_bn=True).astype(np.float32) for m in wl.modules}

    st = [torch.cuda.Stream() for _ in range(K)]
    pipe = ddg.Pipeline(H.descs_for(wl), [s.cuda_stream for s in st])
    if opt == "adam":
        pipe.set_optimizer(ddg.DDG_OPT_ADAM)
    for k in theta:
        pipe.module(k).set_params(theta[k])
    loss_p = torch.zeros(steps, device="cuda")
    torch.cuda.synchronize()
    for t in range(steps):
        pipe.step(*data[t], lr, loss_p[t:t + 1])
    pipe.sync()

    mods = [ddg.Module(d) for d in H.descs_for(wl)]
    for k, m in enumerate(mods, 1):
        if opt == "adam":
            m.set_optimizer(ddg.DDG_OPT_ADAM)
        m.set_params(theta[k])
    sh = [(wl.batch, m.in_h, m.in_w, m.in_c) for m in wl.modules]
    new = lambda k: torch.zeros(sh[k], device="cuda", dtype=H.tdtype(wl))
    mail = [[None] + [new(k) for k in range(1, K)] for _ in range(2)]
    loss_m = torch.zeros(steps, device="cuda")
    for t in range(steps):
        h = data[t][0]
        for k in range(1, K + 1):
            out = new(k) if k < K else None
            torch.cuda.synchronize()
            mods[k - 1].forward(t, h, out)
            mods[k - 1].sync()
            h = out
        for k in range(1, K + 1):
            on = t - K + k >= 0
            mods[k - 1].backward_delayed(t, delta_in=mail[(t - 1) % 2][k] if on and k < K else None, labels=data[t][1] if k == K else None,
                                         delta_out=mail[t % 2][k - 1] if k > 1 else None, loss_out=loss_m[t:t + 1] if k == K else None)
            mods[k - 1].update(t, lr)
            mods[k - 1].sync()
    assert torch.equal(loss_p, loss_m) and bool(torch.isfinite(loss_p).all())
    for k in range(1, K + 1):
        a, b = pipe.module(k), mods[k - 1]
        assert np.array_equal(a.get_params(), b.get_params()) and np.array_equal(a.get_velocity(), b.get_velocity())
        assert np.array_equal(a.get_grad(), b.get_grad())
        b.close()
    pipe.close()
