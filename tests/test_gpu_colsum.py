"""GPU parity of the bias gradients that leave the epilogues of the data gradients: column sums of the masked output, one partial row a pixel
tile, on every tiling of the flat tiles and of the 128-channel tiles, tiles that are cut short among them."""
import numpy as np
import pytest
import torch

from tests.test_gpu_step import _setup

pytestmark = pytest.mark.gpu

FLAT = [114, 118, 122, 124, 128, 132, 134, 142, 144]
# 8 x 28 strips need maps of 28 columns
CASES = [(force, 3, 64) for force in FLAT + [204, 205, 206]] + [(203, 2, 224)]


@pytest.mark.parametrize("force,B,image", CASES)
def test_bias_gradients_of_every_tiling(orc, force, B, image):
    import paper_1811_01532_amd as wap
    want = "conv_tile2d_flat_kernel<%d,%d," % divmod(force - 100, 10) if force < 200 else "conv_tile2d_kernel<1,28,7,1," if force == 203 else "conv_tile2d_kernel<1,0,%d,1," % (force - 200)
    print(f"[case] column sums force={force} B={B} image={image}", flush=True)
    sums = []
    wap.lib().wap_debug_force(force, -1, -1)
    try:
        for flags in (wap.WAP_STEP_STORE_GRADS | wap.WAP_STEP_BIAS, wap.WAP_STEP_KEEP_GRADS | wap.WAP_STEP_BIAS):
            plan, ar, shapes, _, weights, _, _ = _setup("vgg16", B, image, flags, 540)
            ops = plan.ops()
            if not sums:
                fused = [o[0].split(".")[0] for o in ops if "bias_grad" in o[0] and want in o[1]]  # layers whose data gradient sums for the layer below
                assert len(fused) >= 3, ops
            plan.run(ar.buf)
            torch.cuda.synchronize()
            sums.append({d["name"]: ar.f32(d["name"] + ".db", (d["K"],)).double().cpu().numpy() for d in shapes})
    finally:
        wap.lib().wap_debug_force(-1, -1, -1)
    # the kept-gradients plan sums each layer's gradient in a pass of its own (checked against the oracle elsewhere): the same numbers in another order
    for name, a in sums[1].items():
        b = sums[0][name]
        assert np.max(np.abs(a - b)) <= 1e-5 * max(np.max(np.abs(a)), 1e-30), name
        assert np.max(np.abs(a)) > 0
