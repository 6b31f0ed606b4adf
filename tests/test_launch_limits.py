"""The dynamic LDS of every launch lies within what its kernel was given, in whatever order a process makes its calls (no GPU:
seen from the library's calls to the runtime)."""
import pytest

from tests import recorded


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return recorded.build(tmp_path_factory.mktemp("recorder"))


# (N, H, W, C, K, filter side, stride, pad): of one kernel, reductions of one tile and of several
WGRADS = {
    "16-byte loads": [(1, 7, 7, 512, 512, 3, 1, 1), (1, 13, 5, 128, 136, 1, 1, 0)],
    "unaligned loads": [(1, 8, 8, 9, 11, 3, 1, 1), (1, 13, 9, 9, 11, 3, 1, 1)],
    "element by element": [(1, 8, 8, 5, 6, 3, 1, 1), (1, 13, 9, 5, 6, 3, 1, 1)],
}


@pytest.mark.parametrize("which", WGRADS)
@pytest.mark.parametrize("order", [1, -1])
def test_weight_gradient_of_one_tile_first_or_last(so, which, order):
    calls = recorded.launches(recorded.run(so, f"""
m = Mem(1 << 34)
for N, H, W, C, K, R, stride, pad in {WGRADS[which][::order]}:
    wap.wap_conv2d_bwd_weight(wap.conv_desc(N, H, W, C, K, R, R, stride, pad), m, m, m, m, stream=0)
"""))
    main = [c for c in calls if "wgrad_kernel" in c.kernel]
    assert len(main) == 2 and main[0].kernel == main[1].kernel and main[0].smem != main[1].smem
    assert all(c.smem <= c.limit for c in calls), calls
