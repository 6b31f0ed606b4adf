"""Steps whose fully-connected weight gradients run on a second stream beside the convolutions (which launches do: test_step_streams.py):
the same weights as on one stream, as a captured graph runs the list, with several runs in flight at once."""
import threading

import pytest
import torch

from tests.test_gpu_step import _setup

pytestmark = pytest.mark.gpu


def _params(plan, buf):
    off, nb = plan.tensors()["params.w32"]
    return buf[off:off + nb].clone()


# (more rows than the limit, and stored gradients: the list has one stream anyway)
@pytest.mark.parametrize("net,B,image,flags,forks", [("alexnet", 2, 131, 0, True), ("alexnet", 64, 67, 2, True), ("vgg16", 3, 64, 0, True),
                                                     ("alexnet", 5, 67, 2, True), ("alexnet", 65, 67, 0, False), ("alexnet", 3, 67, 6, False)])
def test_beside_is_bitwise_the_same(orc, net, B, image, flags, forks):
    plan, ar, *_ = _setup(net, B, image, flags, 560)
    assert ("workspace2" in plan.tensors()) == forks
    print(f"[case] step beside {net} B={B} image={image} flags={flags}", flush=True)
    start = ar.buf.clone()
    for _ in range(3):
        plan.run(ar.buf)
    torch.cuda.synchronize()
    got = _params(plan, ar.buf)
    ar.buf.copy_(start)
    plan.time(ar.buf, steps=3)
    torch.cuda.synchronize()
    assert torch.equal(got, _params(plan, ar.buf))
    # inside a capture of the caller's the list stays on the caller's stream
    ar.buf.copy_(start)
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        plan.run(ar.buf, stream=side)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
    assert torch.equal(got, _params(plan, ar.buf))


def test_runs_of_one_plan_from_several_threads(orc):
    """One plan, four arenas, a thread and a stream each, more runs in flight than one after the other: every arena ends as a
    run by itself leaves it."""
    plan, ar, *_ = _setup("alexnet", 4, 131, 0, 561)
    assert "workspace2" in plan.tensors()
    print("[case] step beside, four threads", flush=True)
    arenas = [ar.buf.clone() for _ in range(4)]
    for _ in range(6):
        plan.run(ar.buf)
    torch.cuda.synchronize()
    want = _params(plan, ar.buf)
    errors = []

    def work(i):
        try:
            s = torch.cuda.Stream()
            for _ in range(6):
                plan.run(arenas[i], stream=s)
            s.synchronize()
        except Exception as e:  # reported by the test's thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for a in arenas:
        assert torch.equal(_params(plan, a), want)
