"""Which kernel the forced cases of the GPU parity test run, without a GPU: a force that a shape cannot use is ignored, and the case would
then test something else."""
import pytest

from tests.test_gpu_conv import CASES

# data gradients that the forced tiling cannot run (channels of dy that fill no 16-channel step of every wavefront)
NO_FLAT_GRADIENT = {"flat_14_under_one_tile_k40", "flat_22_odd_slices_k72", "flat_42_w14_k136"}
STRIPS, FILL = 203, {204: 4, 205: 5, 206: 6}
PICKED = {  # cases that leave the choice to the shape: what they are there for
    "split_unpacked_forward_w13": ("conv_tile2d_kernel<1,0,2,1,false,true>", None), "split_packed_forward_w14": ("conv_tile2d_kernel<1,0,2,1,false,true>", None),
    "flat_packed_forward_w28": ("conv_tile2d_flat_kernel<", None), "fill_5_picked_w14": ("conv_tile2d_kernel<1,0,5,1,false,true>", "conv_tile2d_flat_kernel<"),
    "c3_groups_1_w138": ("conv_c3_fwd_strided_kernel<2,1>", None), "c3_groups_1_w139_no_border_k32": ("conv_c3_fwd_strided_kernel<1,1>", None),
    "c3_groups_1_low_image_wide_border": ("conv_c3_fwd_strided_kernel<1,1>", None), "c3_groups_2_w226": ("conv_c3_fwd_strided_kernel<2,2>", None),
    "c3_groups_4_k32_cut_short": ("conv_c3_fwd_strided_kernel<1,4>", None), "c3_groups_4_k64": ("conv_c3_fwd_strided_kernel<2,4>", None),
    "flat_picked_5x5_pooled": (None, "conv_tile2d_flat_kernel<2,2,false,5>"),
}


def _names(shape, force):
    import paper_1811_01532_amd as wap
    wap.lib().wap_debug_force(*force)
    try:
        d = wap.conv_desc(*shape)
        return [wap.wap_conv2d_kernel_name(d, p) for p in (wap.WAP_PASS_FWD, wap.WAP_PASS_BWD_DATA)]
    finally:
        wap.lib().wap_debug_force(-1, -1, -1)


@pytest.mark.parametrize("name,shape,force", [c for c in CASES if c[2][0] >= 100 or c[0].startswith("c3_strided_forced")], ids=lambda v: v if isinstance(v, str) else "")
def test_forced_cases_run_what_they_name(name, shape, force):
    fwd, dx = _names(shape, force)
    if force[0] == 8:
        assert fwd == f"conv_c3_fwd_strided_kernel<{shape[4] // 32}>"
    elif force[0] >= 200:
        want = "conv_tile2d_kernel<1,28,7,1,false,true>" if force[0] == STRIPS else f"conv_tile2d_kernel<1,0,{FILL[force[0]]},1,false,true>"
        assert fwd == dx == want
    else:
        fm, ks = divmod(force[0] - 100, 10)
        want = f"conv_tile2d_flat_kernel<{fm},{ks},false,{shape[5]}>"
        assert fwd == want
        assert (dx == want) != (name in NO_FLAT_GRADIENT), dx


@pytest.mark.parametrize("name,shape,force", [c for c in CASES if c[0] in PICKED], ids=lambda v: v if isinstance(v, str) else "")
def test_picked_cases_run_what_they_are_there_for(name, shape, force):
    for got, want in zip(_names(shape, force), PICKED[name]):
        assert want is None or got.startswith(want), got


def test_every_tiling_has_a_case_with_a_pooled_gradient():
    """3x3 and 5x5 (not with eight wavefronts on one reduction), on maps of even sides, where the data gradient runs on the tiling."""
    import paper_1811_01532_amd as wap
    for R, tilings in ((3, (14, 18, 22, 24, 28, 32, 34, 42, 44)), (5, (14, 22, 24, 32, 34, 42, 44))):
        met = set()
        for name, shape, force in CASES:
            d = wap.conv_desc(*shape)
            if force[0] in range(100, 200) and shape[5] == R and d.P % 2 == 0 and d.Q % 2 == 0 and "flat" in _names(shape, force)[1]:
                met.add(force[0] - 100)
        assert met == set(tilings), (R, met)
