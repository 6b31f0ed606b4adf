"""Which streams a step with a second stream uses, seen from the library's calls to the runtime (no GPU)."""
import pytest

from tests import recorded


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return recorded.build(tmp_path_factory.mktemp("recorder"))


def _sides(calls, *callers):
    """For every step of the recorded calls, in order, the stream beside the caller's (None: one stream)."""
    steps = []
    for c in recorded.launches(calls):
        if c.kernel.find("pack_weights_multi") >= 0:
            steps.append(set())
        steps[-1].add(c.stream)
    return [next(iter(s - set(callers)), None) for s in steps]


RUNS = """
plan = wap.StepPlan("alexnet", 8)
n = plan.arena_bytes()
rec.recorder_hold({hold})
for arena, stream in {runs}:
    plan.run(Mem(n, (1 + arena) << 40), stream=stream)
"""


def test_steps_on_independent_streams_share_no_second_stream_in_flight(so):
    """Each of three streams waits for its own work only, whatever is in flight on the others; one arena's steps, which wait
    for each other anyway, keep theirs."""
    calls = recorded.run(so, RUNS.format(hold=1, runs=[(0, 0x10), (1, 0x20), (2, 0x30), (0, 0x10), (1, 0x20), (0, 0x20)]))
    a, b, c, a2, b2, a3 = _sides(calls, "0x10", "0x20", "0x30")
    assert None not in (a, b, c) and len({a, b, c}) == 3
    assert (a2, b2, a3) == (a, b, a)


def test_steps_on_the_default_stream_share_one(so):
    """Whatever their arenas: they follow each other anyway.  A step on another stream has another."""
    a, b, c, d = _sides(recorded.run(so, RUNS.format(hold=1, runs=[(0, 0), (1, 0), (2, 0x20), (3, 0)])), "(nil)", "0x20")
    assert a is not None and a == b == d and c not in (None, a)


def test_a_second_stream_whose_work_is_done_is_used_again(so):
    a, b, c = _sides(recorded.run(so, RUNS.format(hold=0, runs=[(0, 0x10), (1, 0x20), (2, 0x30)])), "0x10", "0x20", "0x30")
    assert a is not None and a == b == c


def test_more_steps_in_flight_than_second_streams_use_one_stream(so):
    sides = _sides(recorded.run(so, RUNS.format(hold=1, runs=[(i, 0x10) for i in range(18)])), "0x10")
    assert len(set(sides[:16])) == 16 and sides[16:] == [None, None]


@pytest.mark.parametrize("net,mb,flags,forks", [("alexnet", 8, 0, True), ("vgg16", 8, 2, True), ("alexnet", 64, 0, True), ("alexnet", 65, 0, False),
                                                ("alexnet", 8, 4, False), ("vgg16", 22, 0, False)])
def test_timed_steps_are_the_steps_that_run(so, net, mb, flags, forks):
    """The same launches on the same streams, with a mask or without."""
    calls = recorded.launches(recorded.run(so, f"""
plan = wap.StepPlan("{net}", {mb}, flags={flags})
assert ("workspace2" in plan.tensors()) == {forks}
mem = Mem(plan.arena_bytes())
plan.run(mem, stream=0x10)
plan.time(mem, stream=0x10)
plan.time(mem, stream=0x10, op_mask=[i % 3 == 0 for i in range(plan.num_ops())])
"""))
    n = len(calls) // 3
    assert calls[:n] == calls[n:2 * n] == calls[2 * n:]
    assert len({c.stream for c in calls}) == (2 if forks else 1)
