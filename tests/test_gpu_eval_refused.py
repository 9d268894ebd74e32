"""A refused evaluation of a pipeline leaves nothing behind: training goes on bit for bit as in a pipeline that was never
evaluated, whether the first module refuses or the last."""
import numpy as np
import pytest

import workloads as wk
from workloads.configs import custom_cifar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_training_goes_on_after_a_refused_evaluation(dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1804_10574_amd as ddg
    from tests import gpu_harness as H
    print(f"case refused evaluation {dtype}", flush=True)
    wl = custom_cifar(1, [1, 2, 3], batch=32, num_classes=10, hw=32, dtype=dtype, name="eval_refused")
    K = wl.K

    def train(evaluate):
        pipe = ddg.Pipeline(H.descs_for(wl), [torch.cuda.Stream().cuda_stream for _ in range(K)])
        for m in wl.modules:
            pipe.module(m.k).set_params(wk.init_module_params(wl, m, perturb_bn=True).astype(np.float32))
        loss = torch.zeros(8, dtype=torch.float32, device="cuda")
        scratch = torch.zeros(1, dtype=torch.float32, device="cuda")
        for t in range(8):
            x, y = wk.minibatch(wl, t)
            xd, yd = H.to_dev_nhwc(x, wl), torch.from_numpy(y).to("cuda")
            torch.cuda.synchronize()
            if evaluate:
                with pytest.raises(ddg.DDGError) as e:
                    pipe.forward_eval(xd, None, scratch)                  # the loss needs labels: the last module refuses
                assert e.value.status == 1
                with pytest.raises(ddg.DDGError) as e:
                    pipe.forward_eval(xd.flatten()[1:], yd, scratch)      # not 16-byte aligned: the first one does
                assert e.value.status == 1
            pipe.step(xd, yd, 0.05, loss[t:t + 1])
        pipe.sync()
        out = [loss.cpu().numpy()] + [pipe.module(k).get_params() for k in range(1, K + 1)]
        pipe.close()
        return out
    for a, b in zip(train(True), train(False)):
        assert np.array_equal(a, b)
