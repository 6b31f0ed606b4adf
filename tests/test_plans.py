"""CPU-only checks of what a plan promises its caller: which calls need no scratch tensor, which need no workspace."""
import pytest

from tests import recorded


@pytest.fixture(scope="module")
def wap():
    import paper_1811_01532_amd as w
    w.lib()
    return w


@pytest.mark.parametrize("N,H,W,C,K,pad", [(12, 12, 14, 256, 32, 2), (28, 18, 18, 64, 32, 2), (28, 18, 18, 64, 64, 2), (4, 24, 24, 256, 64, 2),
                                           (28, 24, 26, 64, 64, 2), (20, 24, 26, 128, 64, 2), (1, 48, 48, 256, 32, 2), (70, 20, 20, 64, 64, 0)])
def test_pooled_5x5_data_gradients_need_no_scratch_tensor(wap, N, H, W, C, K, pad):
    """Even 5x5 maps on tiles of whole patches: the gradient of the pooled output is routed while the patch is staged."""
    assert wap.wap_conv2d_bwd_pool2x2_fused(wap.conv_desc(N, H, W, C, K, 5, 5, 1, pad), wap.WAP_PASS_BWD_DATA)


# Calls that took no workspace go on without one: unsplit products of the generic kernel, whatever other tiles there are, and forward streams
# whose rows of weights are shorter than 256 KB or that have more than 128 work-groups of 16 features.
FORWARD = [(1, 105, 105, 960, 168, 5, 5, 1, 2), (69, 35, 35, 576, 64, 5, 5, 1, 2), (27, 60, 60, 64, 96, 3, 3, 1, 1),
           (20, 57, 57, 64, 96, 3, 3, 1, 1), (6, 51, 51, 256, 448, 5, 5, 1, 2), (7, 68, 68, 64, 96, 3, 3, 1, 1), (12, 1, 1, 4096, 1000, 1, 1, 1, 0)]
BACKWARD = [(15, 37, 37, 96, 256, 3, 3, 1, 1), (2, 40, 49, 1024, 64, 5, 5, 1, 2), (14, 46, 46, 368, 608, 3, 3, 1, 0),
            (12, 16, 16, 512, 32, 3, 3, 1, 1), (10, 50, 50, 256, 96, 5, 5, 1, 0)]
FC = [(12, 4096, 1000), (11, 4096, 512), (10, 7424, 500), (15, 4096, 11), (6, 5184, 1000), (16, 8128, 256), (4, 25088, 2064)]


@pytest.mark.parametrize("shape", FORWARD)
def test_forward_convolutions_ask_for_no_workspace(wap, shape):
    """With a workspace, without one and on the static array the kernels are the same, so the plan is the one that needs none."""
    assert wap.wap_conv2d_workspace_bytes(wap.conv_desc(*shape), wap.WAP_PASS_FWD) == 0


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return recorded.build(tmp_path_factory.mktemp("recorder"))


def test_data_gradients_run_without_a_workspace_and_better_with_it(so):
    calls = recorded.launches(recorded.run(so, f"""
m = Mem(1 << 34)
for shape in {BACKWARD}:
    d = wap.conv_desc(*shape)
    wap.wap_conv2d_bwd_data(d, m, m, m, None, stream=0)
    wap.wap_conv2d_bwd_data_relu(d, m, m, m, m, None, stream=0)
    if shape[1] % 2 == 0 and shape[2] % 2 == 0 and d.P % 2 == 0:
        wap.wap_conv2d_bwd_data_pool2x2(d, m, m, m, m, m, m, None, stream=0)
"""))
    assert all("igemm_kernel" in c.kernel or "maxpool_bwd" in c.kernel for c in calls), calls
    calls = recorded.launches(recorded.run(so, f"""
for shape in {BACKWARD}:
    d = wap.conv_desc(*shape)
    m = Mem(1 << 34)
    wap.wap_conv2d_bwd_data(d, m, m, m, Mem(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA)), stream=0)
"""))
    assert sum("conv_tile2d_flat_kernel" in c.kernel for c in calls) >= 2, calls


def test_fully_connected_calls_run_without_a_workspace_and_divided_with_it(so):
    for ws, launches in (("None", 1), ("Mem(need)", 2)):
        calls = recorded.launches(recorded.run(so, f"""
for shape in {FC}:
    d = wap.fc_desc(*shape)
    m, need = Mem(1 << 34), wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD)
    wap.wap_fc_fwd(d, m, m, None, m, {ws}, stream=0)
"""))
        assert sum("fc_fwd_kernel" in c.kernel for c in calls) == len(FC)
        assert len(calls) > len(FC) if launches == 2 else len(calls) == len(FC), calls


def test_odd_features_divide_the_reduction_where_the_rows_are_long(wap):
    """9216 -> 1438 in halves takes 12.6 us, by eight features without a second launch 13.6; short rows gain nothing from fewer features."""
    for B, n_in, n_out in ((6, 9216, 1438), (5, 9216, 1787), (7, 9216, 1601), (7, 8304, 1653)):
        assert wap.wap_fc_workspace_bytes(wap.fc_desc(B, n_in, n_out), wap.WAP_PASS_FWD) == 2 * 4 * B * n_out


def test_streamed_weight_gradients_by_shape(wap):
    """Fully-connected weight gradients as streams of the weights only where these are no slower than the tiles: not the largest even
    shapes, weight rows that end in the middle of a line, long rows of few outputs, or many batch rows of a large layer."""
    def streams(B, n_in, n_out):
        return wap.wap_conv2d_kernel_name(wap.conv_desc(B, 1, 1, n_in, n_out, 1, 1, 1, 0), wap.WAP_PASS_BWD_WEIGHT) == "fc_dw_kernel"
    for c in ((8, 9216, 4096), (32, 4096, 4096), (20, 25088, 1000), (64, 9216, 4096), (48, 4096, 512), (96, 4096, 500), (8, 4504, 512),
              (100, 2052, 333), (2, 25088, 4097)):
        assert streams(*c), c
    for c in ((20, 25088, 4096), (40, 9216, 512), (33, 9216, 104), (2, 4504, 4096), (3, 8856, 4096), (83, 9216, 232), (40, 4096, 1000), (100, 9216, 500), (80, 4096, 2036), (64, 25088, 10)):
        assert not streams(*c), c


@pytest.mark.parametrize("minibatch,store", [(8, False), (22, True), (32, True)])
def test_a_step_streams_its_largest_weight_gradient(wap, minibatch, store):
    """Behind and beside other kernels the stream is ahead or level where the single call is not."""
    ops = {o[0]: o for o in wap.StepPlan("vgg16", minibatch, flags=wap.WAP_STEP_STORE_GRADS if store else 0).ops()}
    assert "fc_dw_kernel" in next(o for n, o in ops.items() if n.startswith("fc6.dW"))


# (shape, pass) of single calls, us on the larger tiles / on the flat tiles that had replaced them
LARGER_TILES = [((10, 63, 63, 64, 128, 3, 3, 1, 1), 1), ((121, 55, 6, 800, 64, 3, 3, 1, 1), 0), ((19, 45, 45, 64, 64, 3, 3, 1, 1), 0),  # 16 / 22, 52 / 72, 12.4 / 16.1
                ((116, 8, 36, 64, 32, 3, 3, 1, 1), 1), ((14, 57, 57, 64, 832, 3, 3, 1, 1), 1), ((72, 64, 8, 64, 64, 3, 3, 1, 0), 1),   # 10.6 / 14.9, 58 / 75, 12.3 / 15.9
                ((8, 61, 61, 128, 256, 3, 3, 1, 0), 1), ((90, 23, 20, 288, 64, 5, 5, 1, 0), 0)]                                        # 27 / 33, 37 / 43
FLAT_TILES = [((32, 13, 13, 384, 256, 3, 3, 1, 1), 0), ((22, 14, 14, 512, 512, 3, 3, 1, 1), 0), ((8, 28, 28, 512, 512, 3, 3, 1, 1), 1), ((19, 28, 28, 64, 64, 3, 3, 1, 1), 0)]


def test_layers_keep_the_larger_tiles_where_these_are_faster(wap):
    def flat(shape, p):
        return wap.wap_conv2d_kernel_name(wap.conv_desc(*shape), p).startswith("conv_tile2d_flat_kernel")
    assert not any(flat(*c) for c in LARGER_TILES), [c for c in LARGER_TILES if flat(*c)]
    assert all(flat(*c) for c in FLAT_TILES), [c for c in FLAT_TILES if not flat(*c)]


def test_divided_reductions_with_packed_weights_keep_their_splits_where_these_are_faster(so):
    """A step's plans, as the per-layer table runs them: one work-group per few pixels walks a long reduction alone on the flat tiles."""
    def forward(shape):  # (the stand-in runtime has no event to wait for: the table ends behind its first pass)
        return [c.kernel for c in recorded.launches(recorded.run(so, f"""
d = wap.conv_desc(*{shape})
try:
    wap.wap_profile_layer(0, d, [d.N], 0, 1, Mem(1 << 34), stream=0)
except wap.WapError:
    pass
"""))]
    for shape in ((2, 6, 58, 1024, 64, 3, 3, 1, 1), (3, 4, 53, 1024, 128, 3, 3, 1, 1), (2, 8, 8, 928, 64, 5, 5, 1, 2), (1, 10, 10, 960, 128, 5, 5, 1, 2)):
        k = forward(shape)      # us, divided / flat: 14.5 / 36, 12.7 / 37, 12.4 / 54, 13 / 65
        assert any("conv_tile2d" in n for n in k) and not any("flat" in n for n in k), (shape, k)
    assert any("flat" in n for n in forward((8, 14, 14, 512, 512, 3, 3, 1, 1)))


@pytest.mark.parametrize("shape", [(6, 106, 10, 384, 32, 3, 3, 1, 1), (59, 28, 6, 256, 32, 3, 3, 1, 1), (13, 14, 14, 1024, 32, 3, 3, 1, 1), (8, 16, 26, 640, 32, 3, 3, 1, 1)])
def test_one_slice_of_channels_keeps_its_short_tiles(wap, shape):
    assert wap.wap_conv2d_kernel_name(wap.conv_desc(*shape), wap.WAP_PASS_BWD_DATA) == "conv_tile2d_kernel<1,0,2,1,false,true>"


def test_four_features_without_a_second_launch_where_they_fill_the_chip(wap):
    """4096 -> 1000 at 8 rows: 250 work-groups of four features, 7.4 us, not 252 of sixteen over quarters of the reduction, 9."""
    assert wap.wap_fc_workspace_bytes(wap.fc_desc(8, 4096, 1000), wap.WAP_PASS_FWD) == 0


def test_calls_run_in_the_workspace_they_always_took(so):
    """One workspace for the largest minibatch serves the smaller ones, whose deeper splits would ask for more: the last, shorter batch."""
    calls = recorded.launches(recorded.run(so, """
m = Mem(1 << 34)
largest = wap.wap_conv2d_workspace_bytes(wap.conv_desc(100, 15, 15, 64, 32, 3, 3, 1, 0), wap.WAP_PASS_BWD_WEIGHT)
d = wap.conv_desc(64, 15, 15, 64, 32, 3, 3, 1, 0)
assert largest < wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT)
w = Mem(largest)
wap.wap_conv2d_bwd_weight(d, m, m, m, w, stream=0)
wap.wap_conv2d_bwd_weight_sgd(d, m, m, m, m, 0.1, m, w, stream=0)
wap.wap_fc_fwd(wap.fc_desc(7, 25088, 500), m, m, None, m, Mem(6 * 4 * 7 * 500), stream=0)
wap.wap_fc_fwd(wap.fc_desc(1, 9216, 512), m, m, None, m, Mem(2 * 4 * 512), stream=0)
"""))
    assert sum("wgrad_kernel" in c.kernel for c in calls) == 2 and sum("fc_fwd_kernel" in c.kernel for c in calls) == 2, calls


# (inputs, outputs) with row counts whose query is less than what the generic product of fewer rows takes
ROWS = [(1344, 500), (1088, 572), (1152, 500), (1088, 1000), (1472, 500), (1216, 512), (1536, 240), (2112, 512), (2816, 517), (6080, 1351), (4675, 616)]


def test_a_workspace_for_more_rows_serves_fewer(so):
    """Fully-connected forward passes of 17 to 64 rows in the workspace that the query gives for a larger count: the last, shorter batch.
    Without any, layers whose larger counts all need one are refused as they are at those."""
    recorded.run(so, f"""
m = Mem(1 << 34)
for i, o in {ROWS}:
    need = {{n: wap.wap_fc_workspace_bytes(wap.fc_desc(n, i, o), wap.WAP_PASS_FWD) for n in range(17, 65)}}
    for most in range(18, 65):
        if any(need[n] > need[most] for n in range(17, most)):
            for n in range(17, most):
                wap.wap_fc_fwd(wap.fc_desc(n, i, o), m, m, None, m, Mem(need[most]) if need[most] else None, stream=0)
for n in range(17, 65):
    for ws in (None, Mem(1024)):
        try:
            wap.wap_fc_fwd(wap.fc_desc(n, 25088, 4096), m, m, None, m, ws, stream=0)
        except wap.WapError as e:
            assert e.status == wap.WAP_EWORKSPACE
        else:
            raise AssertionError(n)
""")


@pytest.mark.parametrize("H,W,K", [(14, 64, 32), (8, 32, 64), (16, 32, 64), (32, 32, 32), (20, 96, 64), (7, 160, 64)])
def test_a_first_layer_workspace_for_more_images_serves_fewer(so, H, W, K):
    """Weight gradient of a 3x3 first layer: below 4096 pixels another kernel takes it, in the workspace for any larger number of images."""
    recorded.run(so, f"""
m = Mem(1 << 34)
first = -(-4096 // {H * W})
for most in range(first, first + 70):
    w = Mem(wap.wap_conv2d_workspace_bytes(wap.conv_desc(most, {H}, {W}, 3, {K}, 3, 3, 1, 1), wap.WAP_PASS_BWD_WEIGHT))
    for n in range(1, most):
        d = wap.conv_desc(n, {H}, {W}, 3, {K}, 3, 3, 1, 1)
        wap.wap_conv2d_bwd_weight(d, m, m, m, w, stream=0)
        wap.wap_conv2d_bwd_weight_sgd(d, m, m, m, m, 0.1, m, w, stream=0)
""")


def test_operands_pass_the_cache_only_where_that_is_faster(so):
    """Elements around the sizes from which single updates and ReLU derivatives take the same time through and past the cache."""
    def once(calls):
        return [c.kernel.split("_kernel")[1].startswith("ILb1E") for c in recorded.launches(recorded.run(so, "m = Mem(1 << 40)\nm2 = Mem(1 << 40, 1 << 41)\n" + calls))]
    assert once("for n in (24, 28, 34, 36, 38, 60): wap.wap_sgd_update(n * 10**6, m, m, 0.1, m, stream=0)") == [False] * 4 + [True] * 2
    assert once("for n in (28, 34, 44, 46, 60): wap.wap_sgd_update(n * 10**6, m, m, 0.1, None, stream=0)") == [False] * 3 + [True] * 2
    assert once("for n in (42, 46, 48, 52, 77): wap.wap_relu_bwd(m, m, m2, n * 10**6, stream=0)") == [False] * 3 + [True] * 2
    assert once("for n in (52, 77, 84, 92): wap.wap_relu_bwd(m, m, m, n * 10**6, stream=0)") == [False] * 3 + [True]


def test_kernels_of_the_forward_stream_cases(so):
    """Every case that the GPU test of two and four blocks of rows runs, with the workspace it gives: the stream in its four forms, or the
    generic kernel where the line to it is meant."""
    from tests.test_gpu_fc_rows import CASES, SHORT
    assert {c[3] for c in CASES} == {None, (True, 2), (False, 2), (True, 4), (False, 4)}
    for case in CASES + SHORT:
        calls = recorded.launches(recorded.run(so, f"""
m, d = Mem(1 << 34), wap.fc_desc(*{case[:3]})
need = {case[3] if case in SHORT else "wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD)"}
wap.wap_fc_fwd(d, m, m, None, m, Mem(need) if need else None, stream=0)
"""))
        want = (case[1] % 8 == 0, 2 if case[0] <= 32 else 4) if case in SHORT else case[3]
        assert ("igemm_kernel" if want is None else "fc_fwd_kernelILb%dELi%dE" % want) in calls[0].kernel, (case, calls)
        assert len(calls) == 1 or case not in SHORT


def test_stored_gradients_of_the_step_cases_pass_the_cache(so):
    """The kernels behind the GPU test of stored gradients: the stream and the generic tiles in the form that passes the cache."""
    from tests.test_gpu_past_cache import STEPS
    for net, B, image in STEPS:
        names = [c.kernel for c in recorded.launches(recorded.run(so, f"""
p = wap.StepPlan("{net}", {B}, image={image}, flags=wap.WAP_STEP_STORE_GRADS)
p.run(Mem(p.arena_bytes()), stream=0x10)
"""))]
        want = "Lb0ELb1EEE" if B <= 64 else "ILi128ELi128ELi2ELi2ELi0ELb1EEE"
        assert any(("fc_dw_kernel" if B <= 64 else "wgrad_kernel") in n and want in n for n in names), (net, B, names)


def test_work_groups_of_the_streams(so):
    """4096 work-groups walk where that is the faster way: conversions to 63 M elements, updates and ReLU derivatives to 1.5 x 2^20 vectors,
    max-pools of channel counts that are no multiple of 8.  Everything else has a thread for each item."""
    def groups(calls):
        return [c.groups for c in recorded.launches(recorded.run(so, "m = Mem(1 << 40)\nm2 = Mem(1 << 40, 1 << 41)\n" + calls))]
    M = 10 ** 6
    assert groups(f"for n in (1000, 4 * {M}, 10 * {M}, 62 * {M}, 64 * {M}): wap.wap_cast_f32_bf16(n, m, m2, stream=0)") == [1, 3907, 4096, 4096, 62501]
    assert groups(f"for n in (1000, 8 * {M}, 12 * {M}, 13 * {M}, 80 * {M}): wap.wap_relu_bwd(m, m, m2, n, stream=0)") == [1, 3907, 4096, 6348, 39063]
    assert groups(f"for n in (1000, 4 * {M}, 6 * {M}, 7 * {M}, 80 * {M}): wap.wap_sgd_update(n, m, m, 0.1, m2, stream=0)") == [1, 3907, 4096, 6836, 78125]
    for C, want in ((44, 4096), (48, 256 * 35 * 35 * 6 // 256)):
        assert groups(f"""
wap.wap_maxpool_fwd(256, 70, 70, {C}, 2, 2, m, m2, m, stream=0)
wap.wap_maxpool_bwd(256, 70, 70, {C}, 2, 2, m, m, m, m2, stream=0)
""") == [want] * 2


def test_odd_rows_stream_only_where_that_is_faster(so):
    """17 to 64 rows of odd length: beside what the GPU test runs, layers that were timed on either side of the line, and the next even length."""
    def stream(B, i, o):
        calls = recorded.launches(recorded.run(so, f"""
m, d = Mem(1 << 34), wap.fc_desc({B}, {i}, {o})
need = wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD)
wap.wap_fc_fwd(d, m, m, None, m, Mem(need) if need else None, stream=0)
"""))
        return "fc_fwd_kernel" in calls[0].kernel
    assert [stream(*c) for c in ((47, 4789, 4096), (64, 6133, 1000), (49, 3353, 4096), (52, 21501, 500), (32, 17215, 1000))] == [False] * 5
    assert [stream(*c) for c in ((33, 7283, 500), (41, 7611, 9), (40, 693, 512), (21, 5991, 512), (47, 4790, 4096), (64, 6132, 1000), (52, 21502, 500))] == [True] * 7


def test_odd_rows_run_in_what_their_stream_takes(so):
    """Layers whose rows of odd length the generic kernel takes run without a workspace, or in that of the stream's partial sums, as well."""
    recorded.run(so, """
m = Mem(1 << 34)
for B, i, o, splits in ((47, 4789, 4096, 1), (49, 3353, 4096, 1), (64, 6133, 1000, 4), (38, 2013, 500, 1), (52, 21501, 500, 7)):
    d = wap.fc_desc(B, i, o)
    have = 4 * splits * B * o if splits > 1 else 0
    assert wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD) > have
    wap.wap_fc_fwd(d, m, m, None, m, Mem(have) if have else None, stream=0)
    c = wap.conv_desc(B, 1, 1, i, o, 1, 1, 1, 0)
    assert wap.wap_conv2d_workspace_bytes(c, wap.WAP_PASS_FWD) == 0 or splits > 1
""")


def test_fully_connected_data_gradients_alone_and_with_sums(so):
    """A call runs the kernel without column sums, the layers of a step with biases the one that leaves them."""
    calls = [c.kernel for c in recorded.launches(recorded.run(so, """
m = Mem(1 << 34)
for B, i, o in ((96, 4096, 500), (8, 9216, 1000), (16, 4100, 333)):
    wap.wap_fc_bwd(wap.fc_desc(B, i, o), m, m, m, m, None, None, stream=0)
p = wap.StepPlan("alexnet", 5, image=99, flags=wap.WAP_STEP_BIAS)
p.run(Mem(p.arena_bytes()), stream=0x10)
""")) if "fc_dx_kernel" in c.kernel]
    assert [("Lb0EEE" in c, "Lb1EEE" in c) for c in calls] == [(True, False)] * 3 + [(False, True)] * 2 + [(True, False)], calls


def test_max_pools_backward_alone_and_with_sums(so):
    """A call runs the kernel without the arguments of column sums and mean loss, the pools of a step with biases the one that has them."""
    calls = [c.kernel for c in recorded.launches(recorded.run(so, """
m = Mem(1 << 34)
for win, C in ((2, 64), (3, 200), (2, 9), (3, 9)):
    wap.wap_maxpool_bwd(31, 19, 19, C, win, 2, m, m, m, m, stream=0)
p = wap.StepPlan("alexnet", 5, image=99, flags=wap.WAP_STEP_BIAS)
p.run(Mem(p.arena_bytes()), stream=0x10)
""")) if "maxpool_bwd" in c.kernel]
    assert all("maxpool_bwd_s2_kernelILi%dELi%dEE" % (v, w) in c for (v, w), c in zip(((8, 2), (8, 3), (1, 2), (1, 3)), calls)), calls
    assert len(calls) == 7 and all("maxpool_bwd_s2_sums_kernelILi3ELb1E" in c for c in calls[4:]), calls


def test_divided_5x5_calls_of_long_reductions(so):
    """Single calls on either side of four pixels a channel: below, the divided reduction of the generic kernel; with up to 256 channels, the flat tiles."""
    printed = {}
    recorded.run(so, """
for N, H, C, K in ((9, 10, 400, 384), (8, 11, 440, 384), (30, 6, 432, 448), (13, 10, 328, 512), (1, 33, 416, 384), (5, 22, 392, 384), (10, 13, 408, 512), (24, 10, 424, 256)):
    print("dx", [N * H * H, K, wap.wap_conv2d_kernel_name(wap.conv_desc(N, H, H, C, K, 5, 5, 1, 2), wap.WAP_PASS_BWD_DATA)])
for N, H, C, K in ((19, 8, 320, 264), (23, 8, 448, 296), (2, 35, 384, 472), (5, 20, 320, 304), (29, 8, 256, 424), (20, 6, 256, 512)):
    print("fwd", [N * H * H, C, wap.wap_conv2d_kernel_name(wap.conv_desc(N, H, H, C, K, 5, 5, 1, 2), wap.WAP_PASS_FWD)])
""", printed)
    for M, channels, name in printed["dx"] + printed["fwd"]:
        assert name.startswith("igemm_kernel" if M < 4 * channels and channels > 256 else "conv_tile2d_flat_kernel"), (M, channels, name)
