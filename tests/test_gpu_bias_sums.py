"""GPU: bias gradients that ride on other operations of a step (fully-connected data gradients, max-pools backward, the gradient of the logits in
the common pair of launches) and the mean loss taken beside a max-pool, against the plan that has an operation for each."""
import numpy as np
import pytest
import torch

from tests.test_gpu_step import _setup

pytestmark = pytest.mark.gpu

# one image to several hundred: one and two streams, both kernels of the data gradients, one row of sums and many, pools of odd and even maps
CASES = [("alexnet", 1, 67), ("alexnet", 3, 224), ("alexnet", 33, 67), ("alexnet", 70, 99), ("alexnet", 130, 67), ("alexnet", 300, 67), ("vgg16", 1, 224),
         ("vgg16", 5, 96), ("vgg16", 129, 32)]


@pytest.mark.parametrize("net,B,image", CASES)
@pytest.mark.parametrize("store", [False, True])
def test_bias_gradients_and_mean_loss(net, B, image, store):
    import paper_1811_01532_amd as wap
    print(f"[case] bias sums {net} B={B} image={image} store={store}", flush=True)
    got = []
    for flags in (wap.WAP_STEP_KEEP_GRADS | wap.WAP_STEP_BIAS, wap.WAP_STEP_BIAS | (wap.WAP_STEP_STORE_GRADS if store else 0)):
        plan, ar, shapes, _, weights, _, _ = _setup(net, B, image, flags, 550)
        names = [o[0] for o in plan.ops()]
        if not flags & wap.WAP_STEP_KEEP_GRADS:
            assert any("pool_relu_bwd+bias_grad" in n for n in names) and "fc8.bias_grad" not in names, names
        plan.run(ar.buf)
        torch.cuda.synchronize()
        got.append(({k: ar.f32(k + ".db", (weights[k].shape[0],)).double().cpu().numpy() for k in weights if not k.endswith("#bias")}, ar.f32("loss", (4,))[0].item()))
    assert got[0][1] == got[1][1] and np.isfinite(got[0][1])
    for name, a in got[0][0].items():  # sums of the same numbers in another order
        b = got[1][0][name]
        assert np.max(np.abs(a - b)) <= 1e-5 * max(np.max(np.abs(a)), 1e-30) and np.max(np.abs(a)) > 0, name
