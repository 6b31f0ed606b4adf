"""Weight gradients of several layers in one launch: every layer's gradient against the fp64 oracle on the device's own
operands, at minibatches whose runs of tiles end inside blocks, on block borders and behind the last tile."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu
from tests.test_gpu_step import _setup

pytestmark = pytest.mark.gpu


# (alexnet 224: three layers of 13 x 13; vgg16 112 / 64: maps of 56, 28 and 14 pixels, layers of 64 .. 512 channels)
@pytest.mark.parametrize("net,B,image", [("alexnet", 1, 224), ("alexnet", 7, 224), ("alexnet", 33, 224), ("vgg16", 1, 112), ("vgg16", 3, 112),
                                         ("vgg16", 5, 64)])
def test_grouped_weight_gradients(orc, net, B, image):
    import paper_1811_01532_amd as wap
    plan, ar, shapes, _, _, xb, _ = _setup(net, B, image, wap.WAP_STEP_KEEP_GRADS, 540)
    grouped = [o[0].split(".")[0] for o in plan.ops() if o[1].startswith("wgrad_patch_group_kernel")]
    print(f"[case] grouped weight gradients {net} B={B} image={image}: {grouped}", flush=True)
    assert len(grouped) >= 2
    plan.run(ar.buf)
    torch.cuda.synchronize()
    x = orc.bf16_bits_to_f64(xb)
    for i, d in enumerate(shapes):
        L = d["name"]
        if L in grouped:
            g = gu.host_f64(ar.bf16("gm." + L + ".y", (B, d["P"], d["Q"], d["K"])))
            ref = orc.conv2d_bwd_weight(x, g, (d["K"], d["R"], d["S"], d["C"]), (d["stride"],) * 2, (d["pad"],) * 2)
            got = gu.host_f64(ar.f32(L + ".dw", ref.shape))
            assert gu.rel_err(got, ref) <= gu.TOL_F32_OUT, L
        o = d["out_hw"]
        x = gu.host_f64(ar.bf16(L + ".pool.y", (B, o, o, d["K"])) if d["pool"] else ar.bf16(L + ".y", (B, d["P"], d["Q"], d["K"])))


def test_the_sums_do_not_depend_on_the_layout(orc):
    """The production plan, which routes pooled gradients in the loaders, and the one that keeps every intermediate group the
    same layers and cut them alike: the same stored gradients, bit for bit."""
    import paper_1811_01532_amd as wap
    res = []
    for flags in (wap.WAP_STEP_KEEP_GRADS, wap.WAP_STEP_STORE_GRADS):
        plan, ar, _, _, weights, _, _ = _setup("vgg16", 3, 112, flags, 541)
        print(f"[case] grouped weight gradients, flags {flags}", flush=True)
        plan.run(ar.buf)
        torch.cuda.synchronize()
        names = [k for k in weights if "." not in k and not k.endswith("#bias")]
        res.append({k: ar.f32(k + ".dw", weights[k].shape).clone() for k in names})
        kernels = {o[1] for o in plan.ops()}
        assert any(k.startswith("wgrad_patch_group_kernel<" + ("true" if flags == wap.WAP_STEP_STORE_GRADS else "false")) for k in kernels), kernels
    for k, v in res[0].items():
        assert torch.equal(v, res[1][k]), k
