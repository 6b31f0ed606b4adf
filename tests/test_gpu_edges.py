"""GPU parity at the sizes where a kernel's layout or a dispatch rule changes: edges of tiles, remainders, the smallest and
largest shapes of a branch, each against the fp64 oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# (rows that are no whole 128-byte lines also in chunks: whole rows side by side, odd numbers of them below each other, chunk
# sums added by groups of splits for any number of columns)
# rows around the limit of one row chunk (16 per thread of 1024: 1024 with 16 vectors side by side, 8192 with two, 256
# with 64 scalars) and of the small work-group (two rows per thread of 256), 16- / 8- / 2-byte vectors, column blocks
# with a ragged end
@pytest.mark.parametrize("rows,cols", [(1024, 128), (1025, 128), (8192, 16), (8193, 16), (32, 500), (33, 500), (3, 4),
                                       (256, 125), (257, 125), (70, 3), (100, 4096), (2000, 136), (1, 12), (9, 500), (512, 475), (513, 475), (513, 72),
                                       (6000, 33), (20000, 17), (3001, 1000), (40000, 3), (2049, 2051), (5000, 1)])
def test_bias_grad_layout_edges(orc, rows, cols):
    import paper_1811_01532_amd as wap
    print(f"[case] bias_grad edges rows={rows} cols={cols}", flush=True)
    gb = si.normal_bf16(si.rng(430, rows % 1000 + cols), (rows, cols))
    gd = gu.dev_bf16(gb)
    ws = gu.workspace(wap.wap_bias_grad_workspace_bytes(rows, cols))
    db = torch.full((cols + 8,), float("nan"), dtype=torch.float32, device="cuda")
    wap.wap_bias_grad(rows, cols, gd, db, ws)
    torch.cuda.synchronize()
    assert torch.isnan(db[cols:]).all()          # nothing beyond the last column is written
    ref = orc.bias_grad(orc.bf16_bits_to_f64(gb))
    # fp32 sums of `rows` values of magnitude one: the error grows like sqrt(rows) * 2^-24 of their scale sqrt(rows)
    scale = max(np.abs(ref).max(), np.sqrt(rows))
    assert np.max(np.abs(gu.host_f64(db[:cols]) - ref)) <= 1e-5 * scale


# gradient w.r.t. an image of 1 .. 4 channels: maps one pixel over / under the 8 x 32 and 16 x 64 tiles, strides in one or
# both directions, filters in one group, in several (rows, and taps of rows longer than 16), several passes of 64 channels
@pytest.mark.parametrize("N,H,W,C,K,R,S,stride,pad", [
    (2, 8, 32, 3, 64, 3, 3, 1, 1), (1, 9, 33, 3, 64, 3, 3, 1, 1), (3, 7, 31, 3, 8, 3, 3, 1, 0), (1, 17, 20, 1, 72, 5, 5, 1, 2),
    (1, 16, 64, 3, 64, 11, 11, 4, 2), (2, 33, 65, 3, 96, 11, 11, 4, 2), (1, 40, 37, 3, 136, 7, 7, 2, 3),
    (1, 12, 50, 2, 16, 3, 5, (1, 2), (1, 2)), (1, 13, 40, 4, 40, 4, 3, (2, 1), (0, 1)), (1, 31, 34, 3, 24, 3, 3, 3, 1),
    (1, 10, 60, 4, 16, 2, 19, 1, (1, 9)), (1, 20, 70, 3, 32, 18, 18, 2, 5), (2, 5, 5, 1, 8, 1, 1, 1, 0), (1, 30, 41, 1, 16, 20, 1, 1, (3, 0)),
])
def test_image_gradient_edges(orc, N, H, W, C, K, R, S, stride, pad):
    import paper_1811_01532_amd as wap
    st = (stride, stride) if isinstance(stride, int) else stride
    pd = (pad, pad) if isinstance(pad, int) else pad
    print(f"[case] image gradient {(N, H, W, C, K, R, S, st, pd)}", flush=True)
    P, Q = si.out_dim(H, pd[0], R, st[0]), si.out_dim(W, pd[1], S, st[1])
    gb, wb = si.normal_bf16(si.rng(440, H * W + K), (N, P, Q, K)), si.he_weight_bf16(si.rng(441, R * S + C), (K, R, S, C))
    d = wap.conv_desc(N, H, W, C, K, R, S, st, pd)
    assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_DATA) == "dgrad_thin_kernel"
    dx = torch.full((N * H * W * C + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    wap.wap_conv2d_bwd_data(d, gu.dev_bf16(gb), gu.dev_bf16(wb), dx,
                            gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA)))
    torch.cuda.synchronize()
    assert torch.isnan(dx[N * H * W * C:]).all()
    ref = orc.conv2d_bwd_data(orc.bf16_bits_to_f64(gb), orc.bf16_bits_to_f64(wb), (N, H, W, C), st, pd)
    e = gu.rel_err(gu.host_f64(dx[:N * H * W * C]).reshape(N, H, W, C), ref)
    assert e <= gu.TOL_BF16_OUT, e           # one bf16 rounding of an fp32 sum


# one row or column of dy: strides up to the largest int mean the same as one past the map
@pytest.mark.parametrize("stride", [(12, 20), (2147483647, 2147483647), (2147483646, 1), (1, 2000000000)])
def test_image_gradient_huge_strides(orc, stride):
    import paper_1811_01532_amd as wap
    N, H, W, C, K, R, S, pad = 2, 6, 9, 3, 16, 3, 3, (1, 1)
    print(f"[case] image gradient, stride {stride}", flush=True)
    P, Q = si.out_dim(H, 1, R, stride[0]), si.out_dim(W, 1, S, stride[1])
    gb, wb = si.normal_bf16(si.rng(445, P * Q), (N, P, Q, K)), si.he_weight_bf16(si.rng(446, 0), (K, R, S, C))
    d = wap.conv_desc(N, H, W, C, K, R, S, stride, pad)
    assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_DATA) == "dgrad_thin_kernel"
    dx = torch.full((N, H, W, C), float("nan"), dtype=torch.bfloat16, device="cuda")
    wap.wap_conv2d_bwd_data(d, gu.dev_bf16(gb), gu.dev_bf16(wb), dx,
                            gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA)))
    torch.cuda.synchronize()
    same = tuple(min(s, 20) for s in stride)
    ref = orc.conv2d_bwd_data(orc.bf16_bits_to_f64(gb), orc.bf16_bits_to_f64(wb), (N, H, W, C), same, pad)
    assert gu.rel_err(gu.host_f64(dx), ref) <= gu.TOL_BF16_OUT


# an infinite weight reaches exactly the pixels that meet its tap at a dy pixel of the image, not those whose tap lies beyond
@pytest.mark.parametrize("N,H,W,C,K,R,S,stride,pad", [
    (1, 9, 33, 3, 64, 3, 3, 1, 1), (2, 7, 31, 3, 8, 3, 3, 1, 0), (1, 17, 20, 1, 72, 5, 5, 1, 2), (1, 33, 65, 3, 96, 11, 11, 4, 2),
    (1, 40, 37, 3, 136, 7, 7, 2, 3), (1, 13, 40, 4, 40, 4, 3, (2, 1), (0, 1)), (1, 31, 34, 3, 24, 3, 3, 3, 1),
    (1, 10, 60, 4, 16, 2, 19, 1, (1, 9)), (1, 20, 70, 3, 32, 18, 18, 2, 5)])
def test_image_gradient_infinite_weight(orc, N, H, W, C, K, R, S, stride, pad):
    import paper_1811_01532_amd as wap
    st = (stride, stride) if isinstance(stride, int) else stride
    pd = (pad, pad) if isinstance(pad, int) else pad
    P, Q = si.out_dim(H, pd[0], R, st[0]), si.out_dim(W, pd[1], S, st[1])
    d = wap.conv_desc(N, H, W, C, K, R, S, st, pd)
    assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_DATA) == "dgrad_thin_kernel"
    dy = torch.ones((N, P, Q, K), dtype=torch.bfloat16, device="cuda")
    ones = np.ones((N, P, Q, K))
    for r, s in ((0, 0), (R - 1, S - 1), (R // 2, 0), (0, S - 1)):
        print(f"[case] image gradient, infinite weight {(N, H, W, C, K, R, S, st, pd, r, s)}", flush=True)
        w, hot = torch.ones((K, R, S, C), dtype=torch.bfloat16, device="cuda"), np.zeros((K, R, S, C))
        w[K - 1, r, s, C - 1] = float("inf")
        hot[K - 1, r, s, C - 1] = 1.0
        dx = torch.zeros((N, H, W, C), dtype=torch.bfloat16, device="cuda")
        wap.wap_conv2d_bwd_data(d, dy, w, dx, gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA)))
        torch.cuda.synchronize()
        got = gu.host_f64(dx)
        touched = orc.conv2d_bwd_data(ones, hot, (N, H, W, C), st, pd) > 0
        assert touched.any() and np.array_equal(np.isposinf(got), touched) and np.isfinite(got[~touched]).all()


# fully-connected products as streams of the weights: one to eight blocks of 16 rows and one row over / under, features
# that end inside a 16-row block, reductions shorter than one step of all wavefronts, longer, ragged (% 32, % 8, odd),
# divided over work-groups (few features, long rows), two and four columns per lane, a last work-group moved back,
# and the first shapes beyond the limits
@pytest.mark.parametrize("B,n_in,n_out", [
    (1, 8, 1), (16, 40, 17), (17, 512, 16), (32, 520, 33), (33, 4096, 500), (64, 4104, 125), (65, 1024, 130), (96, 4096, 500),
    (128, 2048, 1000), (128, 2051, 1023), (8, 25088, 40), (50, 16392, 24), (64, 12288, 72), (3, 12301, 20), (129, 256, 40),
    (5, 67, 9), (16, 64, 8), (16, 9, 7), (32, 6145, 1031), (33, 6144, 1032), (16, 16391, 50), (64, 65, 1024)])
def test_fc_stream_edges(orc, B, n_in, n_out):
    import paper_1811_01532_amd as wap
    print(f"[case] fc stream {(B, n_in, n_out)}", flush=True)
    xb, Wb = si.normal_bf16(si.rng(450, B + n_in), (B, n_in)), si.he_weight_bf16(si.rng(451, n_in + n_out), (n_out, n_in))
    gb = si.normal_bf16(si.rng(452, B + n_out), (B, n_out))
    bias = si.rng(453, n_out).standard_normal(n_out).astype(np.float32)
    x64, W64, g64 = orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(Wb), orc.bf16_bits_to_f64(gb)
    xd, Wd, gd = gu.dev_bf16(xb), gu.dev_bf16(Wb), gu.dev_bf16(gb)
    for relu in (False, True):
        d = wap.fc_desc(B, n_in, n_out, relu=relu)
        ws = gu.workspace(max(wap.wap_fc_workspace_bytes(d, p) for p in (0, 1, 2)))
        y = torch.full((B * n_out + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        wap.wap_fc_fwd(d, xd, Wd, torch.from_numpy(bias).cuda() if relu else None, y, ws)
        torch.cuda.synchronize()
        assert torch.isnan(y[B * n_out:]).all()
        ref = orc.fc_fwd(x64, W64, bias=bias.astype(np.float64) if relu else None, relu=relu)
        e = gu.rel_err(gu.host_f64(y[:B * n_out]).reshape(B, n_out), ref)
        assert e <= gu.TOL_BF16_OUT, e
    dx = torch.full((B * n_in + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    wap.wap_fc_bwd(d, xd, Wd, gd, dx, None, ws)
    torch.cuda.synchronize()
    assert torch.isnan(dx[B * n_in:]).all()
    e = gu.rel_err(gu.host_f64(dx[:B * n_in]).reshape(B, n_in), orc.fc_bwd_data(g64, W64))
    assert e <= gu.TOL_BF16_OUT, e


# the data-gradient stream with the ReLU derivative of the layer below: a 1x1 convolution on a 1x1 map, rows of dx and of the
# mask at every alignment, the last work-group moved back (columns that no work-group divides), two and four columns per lane
@pytest.mark.parametrize("N,C,K", [(20, 67, 41), (3, 64, 8), (32, 4551, 40), (16, 6147, 33), (65, 6145, 24), (128, 101, 1000)])
def test_fc_stream_masked_data_gradient(orc, N, C, K):
    import paper_1811_01532_amd as wap
    print(f"[case] masked data-gradient stream {(N, C, K)}", flush=True)
    d = wap.conv_desc(N, 1, 1, C, K, 1, 1, 1, 0)
    assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_DATA) == "fc_dx_kernel"
    gb, wb = si.normal_bf16(si.rng(457, N + K), (N, 1, 1, K)), si.he_weight_bf16(si.rng(458, C + K), (K, 1, 1, C))
    xb = si.normal_bf16(si.rng(459, N + C), (N, 1, 1, C))
    dx = torch.full((N * C + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    wap.wap_conv2d_bwd_data_relu(d, gu.dev_bf16(gb), gu.dev_bf16(wb), gu.dev_bf16(xb), dx,
                                 gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA)))
    torch.cuda.synchronize()
    assert torch.isnan(dx[N * C:]).all()
    ref = orc.conv2d_bwd_data(orc.bf16_bits_to_f64(gb), orc.bf16_bits_to_f64(wb), (N, 1, 1, C), (1, 1), (0, 0))
    want = np.where(orc.bf16_bits_to_f64(xb) > 0, ref, 0.0)
    assert gu.rel_err(gu.host_f64(dx[:N * C]).reshape(N, 1, 1, C), want) <= gu.TOL_BF16_OUT


# rows of Wt that are no multiple of 8: an infinite weight among the elements that the row's last vector shares with its
# neighbour, in the last vector's own elements and in front of both reaches exactly its own feature, as +-infinity
@pytest.mark.parametrize("B,n_in,n_out", [(5, 67, 9), (16, 9, 7), (1, 8199, 20), (16, 16391, 50), (3, 1020, 17)])
def test_fc_stream_infinite_weight(orc, B, n_in, n_out):
    import paper_1811_01532_amd as wap
    assert wap.wap_conv2d_kernel_name(wap.conv_desc(B, 1, 1, n_in, n_out, 1, 1, 1, 0), wap.WAP_PASS_FWD) == "fc_fwd_kernel"
    x = orc.bf16_bits_to_f64(si.normal_bf16(si.rng(455, B + n_in), (B, n_in)))
    x[x == 0] = 1.0
    W = orc.bf16_bits_to_f64(si.he_weight_bf16(si.rng(456, n_in + n_out), (n_out, n_in)))
    tail = n_in % 8
    for i, col in enumerate(sorted({0, n_in - 8, n_in - tail - 1, n_in - tail, n_in - 1})):
        W[i, col] = np.inf if i % 2 else -np.inf
    xd, Wd = (gu.dev_bf16(si.f32_to_bf16_bits(t.astype(np.float32))) for t in (x, W))
    for relu in (False, True):
        print(f"[case] fc stream, infinite weight {(B, n_in, n_out, relu)}", flush=True)
        d = wap.fc_desc(B, n_in, n_out, relu=relu)
        y = torch.zeros((B, n_out), dtype=torch.bfloat16, device="cuda")
        wap.wap_fc_fwd(d, xd, Wd, None, y, gu.workspace(wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD)))
        torch.cuda.synchronize()
        ref, got = orc.fc_fwd(x, W, relu=relu), gu.host_f64(y)
        inf = np.isinf(ref)
        assert inf.any() and np.array_equal(got[inf], ref[inf])
        assert gu.rel_err(np.where(inf, 0.0, got), np.where(inf, 0.0, ref)) <= gu.TOL_BF16_OUT


# max-pool: odd / even maps (a last row or column that no window covers, blocks of two input pixels with one inside),
# channels in vectors and one by one, stride 2 with windows of 2 and 3, other strides and windows
@pytest.mark.parametrize("N,H,W,C,win,st", [
    (2, 13, 13, 8, 3, 2), (1, 14, 15, 24, 3, 2), (3, 12, 9, 16, 2, 2), (1, 11, 16, 475, 3, 2), (2, 7, 7, 5, 2, 2), (1, 3, 3, 8, 3, 2),
    (1, 2, 3, 8, 2, 2), (1, 10, 11, 8, 3, 1), (1, 10, 13, 3, 3, 3), (1, 9, 9, 16, 5, 2), (2, 8, 8, 8, 1, 2), (1, 16, 17, 6, 15, 1)])
def test_maxpool_edges(orc, N, H, W, C, win, st):
    import paper_1811_01532_amd as wap
    print(f"[case] maxpool edges {(N, H, W, C, win, st)}", flush=True)
    g = si.rng(460, H * W + C + win)
    x = np.round(g.standard_normal((N, H, W, C)).astype(np.float32) * 4) / 4      # ties, negative windows
    x[0, 0, 0, 0] = -np.inf
    xb = si.f32_to_bf16_bits(x)
    P, Q = si.out_dim(H, 0, win, st), si.out_dim(W, 0, win, st)
    gb = si.normal_bf16(g, (N, P, Q, C))
    n, no = N * H * W * C, N * P * Q * C
    y = torch.full((no + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    am = torch.full((no + 8,), 77, dtype=torch.uint8, device="cuda")
    wap.wap_maxpool_fwd(N, H, W, C, win, st, gu.dev_bf16(xb), y, am)
    x64, g64 = orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(gb)
    yref, amref = orc.maxpool_fwd(x64, win, st)
    torch.cuda.synchronize()
    assert torch.isnan(y[no:]).all() and (am[no:] == 77).all()
    assert np.array_equal(gu.host_f64(y[:no]).reshape(N, P, Q, C), yref)
    assert np.array_equal(am[:no].cpu().numpy().reshape(N, P, Q, C), amref)
    for ry in (None, y):
        dx = torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        wap.wap_maxpool_bwd(N, H, W, C, win, st, gu.dev_bf16(gb), am, ry, dx)
        torch.cuda.synchronize()
        assert torch.isnan(dx[n:]).all()
        ref = orc.maxpool_bwd(g64 if ry is None else np.where(yref > 0, g64, 0.0), amref, (N, H, W, C), win, st)
        assert gu.rel_err(gu.host_f64(dx[:n]).reshape(N, H, W, C), ref) <= gu.TOL_BF16_OUT


# few input channels (1 .. 4): one tile and ragged ones in both directions, filters with an even and an odd side, one to
# sixteen blocks of filter taps, strides and pads in one or both directions, output channels in one block, a part of one,
# several and divided over work-groups, an odd number of elements per image row; several tiles per work-group
@pytest.mark.parametrize("N,H,W,C,K,R,S,stride,pad", [
    (1, 4, 32, 3, 16, 3, 3, 1, 1), (2, 9, 33, 3, 8, 3, 3, 1, 1), (1, 11, 31, 3, 96, 3, 3, 1, 0), (1, 13, 29, 1, 24, 5, 5, 2, 2),
    (2, 35, 35, 3, 40, 11, 11, 4, 2), (1, 47, 47, 3, 96, 7, 7, 2, 3), (1, 12, 50, 2, 16, 3, 5, (1, 2), (1, 2)),
    (1, 13, 40, 4, 40, 4, 3, (2, 1), (0, 1)), (3, 31, 34, 3, 72, 3, 3, 3, 1), (1, 10, 60, 4, 16, 2, 19, 1, (1, 9)),
    (1, 30, 41, 1, 128, 20, 1, 1, (3, 0)), (1, 5, 5, 3, 200, 1, 2, 1, 0), (40, 60, 70, 3, 16, 3, 3, 1, 1), (1, 3, 200, 3, 32, 1, 9, 1, (0, 4)),
    # 768 tiles: two and three channel blocks per work-group in the forward kernel (from 512), the third partly filled; two
    # and three blocks in the weight gradient with three or four and five to eight blocks of filter taps
    (16, 62, 66, 3, 64, 3, 3, 1, 1), (16, 62, 66, 3, 72, 3, 3, 1, 1), (2, 30, 33, 3, 96, 5, 5, 1, 2), (2, 30, 33, 3, 64, 5, 5, 1, 2),
    (1, 30, 33, 3, 64, 7, 7, 1, 3)])
def test_few_channel_edges(orc, N, H, W, C, K, R, S, stride, pad):
    import paper_1811_01532_amd as wap
    st = (stride, stride) if isinstance(stride, int) else stride
    pd = (pad, pad) if isinstance(pad, int) else pad
    print(f"[case] few channels {(N, H, W, C, K, R, S, st, pd)}", flush=True)
    P, Q = si.out_dim(H, pd[0], R, st[0]), si.out_dim(W, pd[1], S, st[1])
    xb, wb = si.normal_bf16(si.rng(470, H * W + K), (N, H, W, C)), si.he_weight_bf16(si.rng(471, R * S + C), (K, R, S, C))
    gb = si.normal_bf16(si.rng(472, H * W + K), (N, P, Q, K))
    bias = si.rng(473, K).standard_normal(K).astype(np.float32)
    x64, w64, g64 = orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(wb), orc.bf16_bits_to_f64(gb)
    xd, ny, nw = gu.dev_bf16(xb), N * P * Q * K, K * R * S * C
    wap.lib().wap_debug_force(15, 7, -1)
    try:
        for relu in (False, True):
            d = wap.conv_desc(N, H, W, C, K, R, S, st, pd, relu=relu)
            assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_FWD) == "conv_thin_fwd_kernel"
            y = torch.full((ny + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
            wap.wap_conv2d_fwd(d, xd, gu.dev_bf16(wb), torch.from_numpy(bias).cuda() if relu else None, y, None)
            torch.cuda.synchronize()
            assert torch.isnan(y[ny:]).all()
            ref = orc.conv2d_fwd(x64, w64, st, pd, bias=bias.astype(np.float64) if relu else None, relu=relu)
            assert gu.rel_err(gu.host_f64(y[:ny]).reshape(N, P, Q, K), ref) <= gu.TOL_BF16_OUT
        assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_WEIGHT) == "wgrad_thin_kernel"
        dw = torch.full((nw + 8,), float("nan"), dtype=torch.float32, device="cuda")
        wap.wap_conv2d_bwd_weight(d, xd, gu.dev_bf16(gb), dw, gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT)))
        torch.cuda.synchronize()
        assert torch.isnan(dw[nw:]).all()
        ref = orc.conv2d_bwd_weight(x64, g64, (K, R, S, C), st, pd)
        assert gu.rel_err(gu.host_f64(dw[:nw]).reshape(K, R, S, C), ref) <= gu.TOL_F32_OUT
        # an infinite pixel reaches exactly the outputs and the weight taps whose receptive field holds it
        xi = x64.copy()
        xi[0, H // 2, W - 1, C - 1] = np.inf
        xid = xd.clone().reshape(N, H, W, C)
        xid[0, H // 2, W - 1, C - 1] = float("inf")
        wap.wap_conv2d_fwd(d, xid, gu.dev_bf16(np.where(wb == 0, 0x3f80, wb).astype(np.uint16)), None, y, None)
        wap.wap_conv2d_bwd_weight(d, xid, torch.ones(N, P, Q, K, dtype=torch.bfloat16, device="cuda"), dw,
                                  gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT)))
        torch.cuda.synchronize()
        touched = orc.conv2d_fwd((~np.isfinite(xi)).astype(np.float64), np.ones((1, R, S, C)), st, pd)[..., 0] > 0
        d0 = gu.host_f64(y[:ny]).reshape(N, P, Q, K)
        assert np.isfinite(d0[~touched]).all()
        taps = orc.conv2d_bwd_weight((~np.isfinite(xi)).astype(np.float64), np.ones((N, P, Q, 1)), (1, R, S, C), st, pd)[0] > 0
        assert np.array_equal(~np.isfinite(gu.host_f64(dw[:nw]).reshape(K, R, S, C)), np.broadcast_to(taps, (K, R, S, C)))
    finally:
        wap.lib().wap_debug_force(-1, -1, -1)


# strided data gradients, one product per phase of the stride: maps that end inside a phase, strides in one or both
# directions, phases without a tap (1x1 filter), more stride than filter, 64 channels or fewer (thin tile), channels in
# vectors and odd, the reduction divided over work-groups, with the ReLU derivative of the layer below, and a stride with
# more phases than the kernel takes
@pytest.mark.parametrize("N,H,W,C,K,R,S,stride,pad,nsplit", [
    (2, 17, 19, 64, 64, 3, 3, 2, 1, -1), (1, 21, 18, 128, 64, 3, 3, 2, 1, -1), (1, 57, 57, 72, 200, 3, 3, 2, 1, -1),
    (2, 14, 15, 24, 40, 1, 1, 2, 0, -1), (1, 12, 13, 40, 64, 5, 5, 2, 2, 2), (1, 16, 11, 16, 24, 4, 3, (2, 1), (1, 0), -1),
    (1, 15, 15, 12, 64, 2, 2, 3, 0, -1), (1, 20, 23, 32, 128, 3, 3, 4, 1, 3), (1, 9, 9, 13, 17, 3, 3, 2, 1, -1),
    (1, 24, 24, 16, 32, 5, 5, 5, 2, -1), (1, 2, 3, 64, 64, 3, 3, 3, 1, -1)])
def test_strided_data_gradient_phases(orc, N, H, W, C, K, R, S, stride, pad, nsplit):
    import paper_1811_01532_amd as wap
    st = (stride, stride) if isinstance(stride, int) else stride
    pd = (pad, pad) if isinstance(pad, int) else pad
    print(f"[case] strided data gradient {(N, H, W, C, K, R, S, st, pd, nsplit)}", flush=True)
    P, Q = si.out_dim(H, pd[0], R, st[0]), si.out_dim(W, pd[1], S, st[1])
    gb, wb = si.normal_bf16(si.rng(480, H * W + K), (N, P, Q, K)), si.he_weight_bf16(si.rng(481, R * S + C), (K, R, S, C))
    xb = si.normal_bf16(si.rng(482, H * W + C), (N, H, W, C))
    d = wap.conv_desc(N, H, W, C, K, R, S, st, pd)
    n = N * H * W * C
    ref = orc.conv2d_bwd_data(orc.bf16_bits_to_f64(gb), orc.bf16_bits_to_f64(wb), (N, H, W, C), st, pd)
    wap.lib().wap_debug_force(-1, -1, nsplit)
    try:
        ws = gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA))
        for mask in (False, True):
            dx = torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
            if mask:
                wap.wap_conv2d_bwd_data_relu(d, gu.dev_bf16(gb), gu.dev_bf16(wb), gu.dev_bf16(xb), dx, ws)
            else:
                wap.wap_conv2d_bwd_data(d, gu.dev_bf16(gb), gu.dev_bf16(wb), dx, ws)
            torch.cuda.synchronize()
            assert torch.isnan(dx[n:]).all()
            want = np.where(orc.bf16_bits_to_f64(xb) > 0, ref, 0.0) if mask else ref
            assert gu.rel_err(gu.host_f64(dx[:n]).reshape(N, H, W, C), want) <= gu.TOL_BF16_OUT
    finally:
        wap.lib().wap_debug_force(-1, -1, -1)


# channel counts that are no multiple of 8, from 8 (the least for unaligned 16-byte loads) up: every remainder, one group and
# many, tiles that end inside a group, one pass only odd, each with the update fused behind the weight gradient, and channel
# counts below 8 (element by element)
@pytest.mark.parametrize("N,H,W,C,K,R,S,stride,pad,nsplit", [
    (1, 9, 8, 9, 8, 3, 3, 1, 1, -1), (2, 7, 7, 15, 23, 3, 3, 1, 1, -1), (1, 6, 5, 12, 20, 3, 3, 1, 1, 1), (1, 13, 11, 119, 64, 3, 3, 1, 1, -1),
    (1, 10, 10, 64, 475, 1, 1, 1, 0, -1), (1, 9, 9, 13, 17, 3, 3, 2, 1, -1), (1, 8, 8, 8, 10, 3, 3, 1, 1, 2), (1, 5, 5, 11, 8, 2, 2, 1, 0, -1),
    (1, 6, 6, 137, 131, 3, 3, 1, 1, 3), (3, 5, 4, 14, 129, 1, 3, 1, (0, 1), -1), (1, 6, 7, 7, 18, 3, 3, 1, 1, -1), (1, 6, 7, 18, 5, 3, 3, 1, 1, -1)])
def test_odd_channel_edges(orc, N, H, W, C, K, R, S, stride, pad, nsplit):
    import paper_1811_01532_amd as wap
    st = (stride, stride) if isinstance(stride, int) else stride
    pd = (pad, pad) if isinstance(pad, int) else pad
    print(f"[case] odd channels {(N, H, W, C, K, R, S, st, pd, nsplit)}", flush=True)
    P, Q = si.out_dim(H, pd[0], R, st[0]), si.out_dim(W, pd[1], S, st[1])
    xb, wb = si.normal_bf16(si.rng(490, H * W + C), (N, H, W, C)), si.he_weight_bf16(si.rng(491, R * S + C), (K, R, S, C))
    gb = si.normal_bf16(si.rng(492, H * W + K), (N, P, Q, K))
    x64, w64, g64 = orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(wb), orc.bf16_bits_to_f64(gb)
    xd, wd, gd = gu.dev_bf16(xb), gu.dev_bf16(wb), gu.dev_bf16(gb)
    d = wap.conv_desc(N, H, W, C, K, R, S, st, pd)
    nx, ny, nw = N * H * W * C, N * P * Q * K, K * R * S * C
    wap.lib().wap_debug_force(-1, -1, nsplit)
    try:
        ws = gu.workspace(max(wap.wap_conv2d_workspace_bytes(d, p) for p in (0, 1, 2)))
        y = torch.full((ny + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        dx = torch.full((nx + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        dw = torch.full((nw + 8,), float("nan"), dtype=torch.float32, device="cuda")
        wap.wap_conv2d_fwd(d, xd, wd, None, y, ws)
        wap.wap_conv2d_bwd_data(d, gd, wd, dx, ws)
        wap.wap_conv2d_bwd_weight(d, xd, gd, dw, ws)
        torch.cuda.synchronize()
        assert torch.isnan(y[ny:]).all() and torch.isnan(dx[nx:]).all() and torch.isnan(dw[nw:]).all()
        assert gu.rel_err(gu.host_f64(y[:ny]).reshape(N, P, Q, K), orc.conv2d_fwd(x64, w64, st, pd)) <= gu.TOL_BF16_OUT
        assert gu.rel_err(gu.host_f64(dx[:nx]).reshape(N, H, W, C), orc.conv2d_bwd_data(g64, w64, (N, H, W, C), st, pd)) <= gu.TOL_BF16_OUT
        assert gu.rel_err(gu.host_f64(dw[:nw]).reshape(K, R, S, C), orc.conv2d_bwd_weight(x64, g64, (K, R, S, C), st, pd)) <= gu.TOL_F32_OUT
        w32 = torch.arange(nw, dtype=torch.float32, device="cuda") / nw
        want = torch.empty_like(w32).copy_(w32)
        wbf, wbf_want = torch.zeros(nw, dtype=torch.bfloat16, device="cuda"), torch.zeros(nw, dtype=torch.bfloat16, device="cuda")
        wap.wap_sgd_update(nw, want, dw[:nw].clone(), 0.5, wbf_want)
        wap.wap_conv2d_bwd_weight_sgd(d, xd, gd, w32, wbf, 0.5, torch.empty(nw, dtype=torch.float32, device="cuda"), ws)
        torch.cuda.synchronize()
        assert torch.equal(w32, want) and torch.equal(wbf, wbf_want)
    finally:
        wap.lib().wap_debug_force(-1, -1, -1)


# the same for fully-connected layers beyond the streaming kernels: odd rows of x, of the weights and of dy
@pytest.mark.parametrize("B,n_in,n_out", [(130, 67, 9), (200, 255, 250), (129, 257, 40), (288, 96, 333), (150, 8, 11), (140, 300, 8)])
def test_odd_fc_edges(orc, B, n_in, n_out):
    import paper_1811_01532_amd as wap
    print(f"[case] odd fc {(B, n_in, n_out)}", flush=True)
    xb, Wb = si.normal_bf16(si.rng(500, B + n_in), (B, n_in)), si.he_weight_bf16(si.rng(501, n_in + n_out), (n_out, n_in))
    gb = si.normal_bf16(si.rng(502, B + n_out), (B, n_out))
    x64, W64, g64 = orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(Wb), orc.bf16_bits_to_f64(gb)
    d = wap.fc_desc(B, n_in, n_out, relu=False)
    ws = gu.workspace(max(wap.wap_fc_workspace_bytes(d, p) for p in (0, 1, 2)))
    y = torch.full((B * n_out + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    dx = torch.full((B * n_in + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((n_out * n_in + 8,), float("nan"), dtype=torch.float32, device="cuda")
    xd, Wd, gd = gu.dev_bf16(xb), gu.dev_bf16(Wb), gu.dev_bf16(gb)
    wap.wap_fc_fwd(d, xd, Wd, None, y, ws)
    wap.wap_fc_bwd(d, xd, Wd, gd, dx, dw, ws)
    torch.cuda.synchronize()
    assert torch.isnan(y[B * n_out:]).all() and torch.isnan(dx[B * n_in:]).all() and torch.isnan(dw[n_out * n_in:]).all()
    assert gu.rel_err(gu.host_f64(y[:B * n_out]).reshape(B, n_out), orc.fc_fwd(x64, W64)) <= gu.TOL_BF16_OUT
    assert gu.rel_err(gu.host_f64(dx[:B * n_in]).reshape(B, n_in), orc.fc_bwd_data(g64, W64)) <= gu.TOL_BF16_OUT
    assert gu.rel_err(gu.host_f64(dw[:n_out * n_in]).reshape(n_out, n_in), g64.T @ x64) <= gu.TOL_F32_OUT


# 5x5 weight gradient on maps whose tiles hold surplus columns and rows: an infinite pixel reaches exactly the taps whose
# receptive field holds it
@pytest.mark.parametrize("H,W,yx", [(27, 27, (26, 26)), (27, 27, (25, 3)), (13, 14, (12, 13)), (9, 31, (8, 30))])
def test_wgrad_5x5_infinite_pixel(orc, H, W, yx):
    import paper_1811_01532_amd as wap
    print(f"[case] 5x5 weight gradient, infinite pixel {(H, W, yx)}", flush=True)
    N, C, K = 2, 64, 32
    d = wap.conv_desc(N, H, W, C, K, 5, 5, 1, 2)
    wap.lib().wap_debug_force(-1, 3, -1)
    try:
        assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_WEIGHT).startswith("wgrad_patch5_kernel")
        x = torch.ones((N, H, W, C), dtype=torch.bfloat16, device="cuda")
        x[1, yx[0], yx[1], 5] = float("inf")
        dw = torch.zeros((K, 5, 5, C), dtype=torch.float32, device="cuda")
        wap.wap_conv2d_bwd_weight(d, x, torch.ones((N, H, W, K), dtype=torch.bfloat16, device="cuda"), dw,
                                  gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT)))
    finally:
        wap.lib().wap_debug_force(-1, -1, -1)
    torch.cuda.synchronize()
    hot = np.zeros((N, H, W, C))
    hot[1, yx[0], yx[1], 5] = 1.0
    taps = orc.conv2d_bwd_weight(hot, np.ones((N, H, W, 1)), (1, 5, 5, C), (1, 1), (2, 2))[0] > 0
    assert np.array_equal(~np.isfinite(gu.host_f64(dw)), np.broadcast_to(taps, (K, 5, 5, C)))
