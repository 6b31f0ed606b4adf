"""GPU parity of the implicit-GEMM kernel where its walk, its wavefront arrangement or its epilogue changes: reduction tiles
around the register sets and the eight of a decoded group, one work-group per CU and more, ragged rows and channels, filters
that divide no tile, the ReLU derivative in the epilogue, each against the fp64 oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# (N, H, W, C, K, R, S, stride, pad): 1 .. 20 reduction tiles in whole slices (C % 64 == 0), in eights and odd; 1 to 600
# work-groups; the last row tile of 1, 32 and 127 pixels; strided (phases) and 1x1 strided (divided taps)
CASES = [
    (1, 5, 5, 64, 72, 1, 1, 1, 0), (1, 8, 16, 128, 128, 1, 1, 1, 0), (1, 3, 43, 192, 136, 1, 1, 1, 0), (1, 11, 23, 320, 65, 1, 1, 1, 0),
    (2, 9, 9, 24, 40, 3, 3, 2, 1), (1, 13, 11, 8, 8, 5, 3, (1, 2), (2, 1)), (1, 20, 20, 72, 200, 3, 3, 2, 1), (3, 14, 14, 56, 24, 7, 7, 1, 3),
    (1, 19, 17, 37, 43, 3, 3, 1, 1), (2, 12, 12, 9, 130, 2, 3, (2, 1), (0, 1)), (1, 15, 15, 119, 33, 3, 3, 2, 1), (1, 7, 7, 5, 6, 3, 3, 1, 1),
    (9, 30, 30, 16, 520, 1, 1, 1, 0), (12, 56, 50, 64, 24, 1, 1, 1, 0), (16, 40, 40, 64, 64, 1, 1, 2, 0), (6, 61, 61, 40, 264, 3, 3, 2, 1),
    (2, 50, 50, 448, 17, 1, 1, 1, 0), (1, 33, 1, 64, 256, 1, 1, 1, 0),
]


@pytest.mark.parametrize("case", CASES)
def test_forward_and_data_gradient(orc, case):
    import paper_1811_01532_amd as wap
    N, H, W, C, K, R, S, stride, pad = case
    st = (stride, stride) if isinstance(stride, int) else stride
    pd = (pad, pad) if isinstance(pad, int) else pad
    print(f"[case] igemm {case}", flush=True)
    P, Q = si.out_dim(H, pd[0], R, st[0]), si.out_dim(W, pd[1], S, st[1])
    xb = si.normal_bf16(si.rng(910, H * W + C), (N, H, W, C))
    wb = si.he_weight_bf16(si.rng(911, R * S + K), (K, R, S, C))
    gb = si.normal_bf16(si.rng(912, P * Q + K), (N, P, Q, K))
    xd, wd, gd = gu.dev_bf16(xb), gu.dev_bf16(wb), gu.dev_bf16(gb)
    x64, w64, g64 = (orc.bf16_bits_to_f64(t) for t in (xb, wb, gb))
    d = wap.conv_desc(N, H, W, C, K, R, S, st, pd)
    y = torch.full((N * P * Q * K + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    bias = torch.arange(K, dtype=torch.float32, device="cuda") * 0.01
    wap.wap_conv2d_fwd(d, xd, wd, bias, y, gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_FWD)))
    torch.cuda.synchronize()
    assert torch.isnan(y[N * P * Q * K:]).all()
    ref = orc.conv2d_fwd(x64, w64, st, pd) + gu.host_f64(bias)
    assert gu.rel_err(gu.host_f64(y[:N * P * Q * K]).reshape(ref.shape), ref) <= gu.TOL_BF16_OUT
    ws = gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA))
    ref = orc.conv2d_bwd_data(g64, w64, (N, H, W, C), st, pd)
    for mask in (False, True):  # x doubles as the activation whose derivative the masked call applies
        dx = torch.full((N * H * W * C + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        if mask:
            wap.wap_conv2d_bwd_data_relu(d, gd, wd, xd, dx, ws)
        else:
            wap.wap_conv2d_bwd_data(d, gd, wd, dx, ws)
        torch.cuda.synchronize()
        assert torch.isnan(dx[N * H * W * C:]).all()
        got = gu.host_f64(dx[:N * H * W * C]).reshape(ref.shape)
        want = np.where(x64 > 0, ref, 0.0) if mask else ref
        assert gu.rel_err(got, want) <= gu.TOL_BF16_OUT, mask
        if mask:
            assert np.all(got[x64 <= 0] == 0)


@pytest.mark.parametrize("B,n_in,n_out", [(17, 64, 100), (33, 512, 1000), (64, 1088, 264), (65, 2048, 500), (129, 640, 4100), (200, 520, 301),
                                          (257, 4096, 129), (70, 8, 3)])
def test_fully_connected(orc, B, n_in, n_out):
    import paper_1811_01532_amd as wap
    print(f"[case] igemm fc {(B, n_in, n_out)}", flush=True)
    xb, wb = si.normal_bf16(si.rng(920, B), (B, n_in)), si.he_weight_bf16(si.rng(921, n_out), (n_out, n_in))
    gb = si.normal_bf16(si.rng(922, B + n_out), (B, n_out))
    xd, wd, gd = gu.dev_bf16(xb), gu.dev_bf16(wb), gu.dev_bf16(gb)
    x64, w64, g64 = (orc.bf16_bits_to_f64(t) for t in (xb, wb, gb))
    d = wap.fc_desc(B, n_in, n_out)
    ws = gu.workspace(max(wap.wap_fc_workspace_bytes(d, p) for p in (wap.WAP_PASS_FWD, wap.WAP_PASS_BWD_DATA)))
    y = torch.empty((B, n_out), dtype=torch.bfloat16, device="cuda")
    dx = torch.empty((B, n_in), dtype=torch.bfloat16, device="cuda")
    wap.wap_fc_fwd(d, xd, wd, None, y, ws)
    wap.wap_fc_bwd(d, xd, wd, gd, dx, None, ws)
    torch.cuda.synchronize()
    assert gu.rel_err(gu.host_f64(y), x64 @ w64.T) <= gu.TOL_BF16_OUT
    assert gu.rel_err(gu.host_f64(dx), g64 @ w64) <= gu.TOL_BF16_OUT


# weight gradient: pixels of 1 .. 9 reduction tiles unsplit and split, both wavefront arrangements, a last tile of one pixel,
# channels in eights, odd and single, columns behind the last tap
@pytest.mark.parametrize("case", [
    (1, 7, 7, 512, 512, 3, 3, 1, 1), (1, 13, 5, 128, 136, 1, 1, 1, 0), (1, 16, 12, 128, 128, 1, 1, 1, 0), (5, 13, 13, 40, 72, 3, 3, 2, 1),
    (2, 16, 18, 24, 40, 5, 5, 1, 2), (3, 19, 17, 37, 43, 3, 3, 1, 1), (1, 9, 9, 9, 257, 3, 3, (2, 1), 1), (4, 20, 20, 64, 64, 3, 3, 2, 1),
    (1, 23, 1, 600, 700, 1, 1, 1, 0), (65, 1, 1, 264, 4100, 1, 1, 1, 0), (193, 1, 1, 520, 301, 1, 1, 1, 0), (1, 8, 8, 5, 6, 3, 3, 1, 1),
    (12, 27, 27, 96, 256, 5, 5, 1, 2),
])
def test_weight_gradient(orc, case):
    import paper_1811_01532_amd as wap
    N, H, W, C, K, R, S, stride, pad = case
    st = (stride, stride) if isinstance(stride, int) else stride
    print(f"[case] wgrad {case}", flush=True)
    P, Q = si.out_dim(H, pad, R, st[0]), si.out_dim(W, pad, S, st[1])
    xb, gb = si.normal_bf16(si.rng(930, H * W + C), (N, H, W, C)), si.normal_bf16(si.rng(931, P * Q + K), (N, P, Q, K))
    d = wap.conv_desc(N, H, W, C, K, R, S, st, (pad, pad))
    n = K * R * S * C
    dw = torch.full((n + 4,), float("nan"), dtype=torch.float32, device="cuda")
    wap.wap_conv2d_bwd_weight(d, gu.dev_bf16(xb), gu.dev_bf16(gb), dw, gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT)))
    torch.cuda.synchronize()
    assert torch.isnan(dw[n:]).all()
    ref = orc.conv2d_bwd_weight(orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(gb), (K, R, S, C), st, (pad, pad))
    assert gu.rel_err(gu.host_f64(dw[:n]).reshape(ref.shape), ref) <= gu.TOL_F32_OUT
