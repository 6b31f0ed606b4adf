"""What a step's launch list says of its operations (no GPU)."""
import pytest

import paper_1811_01532_amd as wap
import synth_inputs as si


def _weights(net, image=224):
    """Elements of every convolution's weights, by layer."""
    return {d["name"]: d["K"] * d["R"] * d["S"] * d["C"] for d in si.conv_shapes(si.NETS[net][0], image)}


@pytest.mark.parametrize("net,mb", [("alexnet", 32), ("vgg16", 64), ("alexnet", 100)])
def test_bytes_of_the_weight_packing(net, mb):
    """The weights of every layer behind the first, whose kernel takes them as they are, for the forward pass and for the
    data gradient: read once and written once as bf16 (no channel count of these layers leaves a block of 32 ragged)."""
    ops = wap.StepPlan(net, mb).ops()
    conv2d = ("conv_tile2d", "conv_tile64", "conv_patch", "conv_wreg")
    first, *rest = _weights(net).items()
    assert all(o[1].startswith(conv2d) for o in ops if o[0].startswith(tuple(n + "." for n, _ in rest)) and ("fwd" in o[0] or "dgrad" in o[0])
               and not o[0].endswith(("pool.fwd", "pool_relu_bwd")))
    assert [o[3] for o in ops if o[0] == "pack_weights"] == [2 * 2 * 2.0 * sum(n for _, n in rest)]
