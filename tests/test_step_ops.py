"""What a step's launch list says of its operations (no GPU)."""
import pytest

import paper_1811_01532_amd as wap
import synth_inputs as si
from tests import recorded


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return recorded.build(tmp_path_factory.mktemp("recorder"))


def _weights(net, image=224):
    """Elements of every convolution's weights, by layer."""
    return {d["name"]: d["K"] * d["R"] * d["S"] * d["C"] for d in si.conv_shapes(si.NETS[net][0], image)}


@pytest.mark.parametrize("net,mb", [("alexnet", 32), ("vgg16", 64), ("alexnet", 100)])
def test_bytes_of_the_weight_packing(net, mb):
    """The weights of every layer behind the first, whose kernel takes them as they are: read once, and written once for the forward pass
    and once for the data gradient, as bf16 (no channel count of these layers leaves a block of 32 ragged)."""
    ops = wap.StepPlan(net, mb).ops()
    conv2d = ("conv_tile2d", "conv_tile64", "conv_patch", "conv_wreg")
    first, *rest = _weights(net).items()
    assert all(o[1].startswith(conv2d) for o in ops if o[0].startswith(tuple(n + "." for n, _ in rest)) and ("fwd" in o[0] or "dgrad" in o[0])
               and not o[0].endswith(("pool.fwd", "pool_relu_bwd")))
    assert [o[3] for o in ops if o[0] == "pack_weights"] == [(1 + 2) * 2.0 * sum(n for _, n in rest)]


def _groups(ops):
    """Runs of operations that share a launch, as lists of indices."""
    out = []
    for i, o in enumerate(ops):
        if o[1].startswith("wgrad_patch_group_kernel"):
            if not o[1].endswith(" (shared)"):
                out.append([])
            out[-1].append(i)
    return out


def test_a_shared_launch_counts_once_and_its_time_is_divided_by_work(so):
    """AlexNet-style and VGG-16, 8 images: as many first operations of a group as group launches, every layer with its own
    FLOPs; of a launch that takes 1000 us (every event pair does here) each layer gets its share, also where a mask asks for
    one layer alone."""
    for net in ("alexnet", "vgg16"):
        plan = wap.StepPlan(net, 8)
        ops, groups = plan.ops(), _groups(plan.ops())
        calls = recorded.run(so, f"""
plan = wap.StepPlan("{net}", 8)
mem = Mem(plan.arena_bytes())
plan.run(mem, stream=0x10)
n = rec.recorder_count()
us, epi = plan.time(mem, stream=0x10)
print("us", us)
print("epi", epi)
for i in {[g[-1] for g in groups]}:
    print("one", plan.time(mem, stream=0x10, op_mask=[k == i for k in range(len(us))])[0])
""", printed=(out := {}))
        run = recorded.launches(calls)[:len(recorded.launches(calls)) // (2 + len(groups))]
        assert groups and sum("wgrad_patch_group_kernel" in c.kernel for c in run) == len(groups)
        assert sum(o[2] for o in ops) == pytest.approx(plan.flops(), rel=1e-12)
        us, epi = out["us"][0], out["epi"][0]
        for g, one in zip(groups, out["one"]):
            assert len(g) >= 2 and g == list(range(g[0], g[-1] + 1))
            whole = sum(ops[i][2] for i in g)
            for i in g:
                assert us[i] == pytest.approx(1000 * ops[i][2] / whole) and epi[i] == pytest.approx(us[i])
            assert one == [pytest.approx(us[i]) if i == g[-1] else 0.0 for i in range(len(ops))]
