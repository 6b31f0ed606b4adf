"""Both packed copies of a step's filters, bit for bit: layers whose copies come from one reading and layers that are packed for one pass only."""
import numpy as np
import pytest
import torch

from tests import gpu_util as gu  # noqa: F401  (skips without a GPU)
from tests.test_gpu_step import _setup

pytestmark = pytest.mark.gpu


def _fragments(m):
    """[n][kk] -> [block of 32][step of 16][half][n % 32][8], zeros past the last n."""
    n, k = m.shape
    m = np.concatenate([m, np.zeros((-n % 32, k), m.dtype)])
    return m.reshape(-1, 32, k // 16, 2, 8).transpose(0, 2, 3, 1, 4).ravel()


@pytest.mark.parametrize("net,B,image", [("vgg16", 2, 32), ("vgg16", 1, 224), ("alexnet", 3, 67), ("alexnet", 40, 224)])
def test_packed_copies_are_the_filters(net, B, image):
    plan, ar, shapes, _, weights, _, _ = _setup(net, B, image, 0, 560)
    print(f"[case] packed weights {net} B={B} image={image}", flush=True)
    plan.run(ar.buf)
    torch.cuda.synchronize()
    seen = {False: 0, True: 0}
    for s in shapes:
        w = weights[s["name"]].view(np.int16)
        K, R, S, C = w.shape
        want = {"fwd": w.reshape(K, -1), "dgrad": w[:, ::-1, ::-1, :].transpose(3, 1, 2, 0).reshape(C, -1)}
        for name in ar.t:
            if not name.startswith("wpack." + s["name"] + "."):
                continue
            back = "dgrad" in name
            got = ar.raw(name).view(torch.int16).cpu().numpy()
            assert np.array_equal(got, _fragments(want["dgrad" if back else "fwd"])), name
            seen[back] += 1
    assert min(seen.values()) >= 2
