"""GPU parity of single convolutions whose divided reduction runs on the flat tiles: the least pixels that do so and one row fewer,
channels past the rule, weights read as they are and packed, channels that are no block of 32, rows of odd length, no padding and more than the filter's half, the ReLU derivative and
a max-pool in the data gradient; filters that outgrow the partial sums' workspace keep the divided plan."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# N, H, W, C, K, filter, padding, forward / data gradient on flat tiles
CASES = [(1, 28, 25, 128, 64, 3, 1, True, True), (1, 27, 25, 128, 64, 3, 1, False, False), (2, 19, 19, 96, 224, 3, 1, True, None), (1, 27, 27, 64, 192, 5, 2, True, None), (2, 27, 27, 64, 192, 5, 2, False, None), (1, 30, 30, 96, 64, 5, 2, False, None), (3, 20, 20, 192, 64, 5, 2, None, True),
         (3, 17, 17, 256, 104, 3, 1, True, None), (3, 21, 17, 104, 256, 3, 0, None, True), (7, 9, 13, 64, 128, 3, 2, True, True), (3, 25, 25, 32, 192, 5, 2, True, None),
         (3, 16, 16, 272, 32, 5, 2, None, True), (4, 30, 30, 160, 224, 3, 1, True, True), (1, 28, 25, 544, 64, 3, 1, False, None), (4, 26, 26, 408, 480, 5, 2, None, False)]


def _flat(wap, d, p):
    return wap.wap_conv2d_kernel_name(d, p).startswith("conv_tile2d_flat")


@pytest.mark.parametrize("N,H,W,C,K,k,pad,fwd,dx", CASES)
def test_single_calls_on_flat_tiles(orc, N, H, W, C, K, k, pad, fwd, dx):
    import paper_1811_01532_amd as wap
    print(f"[case] single flat {(N, H, W, C, K, k, pad)}", flush=True)
    d = wap.conv_desc(N, H, W, C, K, k, k, 1, pad)
    wb = si.he_weight_bf16(si.rng(981, K + C), (K, k, k, C))
    w64, wd = orc.bf16_bits_to_f64(wb), gu.dev_bf16(wb)
    xb, gb = si.normal_bf16(si.rng(982, C), (N, H, W, C)), si.normal_bf16(si.rng(983, K), (N, d.P, d.Q, K))
    x64, g64 = orc.bf16_bits_to_f64(xb), orc.bf16_bits_to_f64(gb)
    xd, gd = gu.dev_bf16(xb), gu.dev_bf16(gb)
    if fwd is not None:
        assert _flat(wap, d, wap.WAP_PASS_FWD) == fwd
        bias = si.rng(984, K).standard_normal(K).astype(np.float32)
        ref = orc.conv2d_fwd(x64, w64, (1, 1), (pad, pad))
        ws = gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_FWD))
        y = torch.full((N * d.P * d.Q * K + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        for relu in (False, True):
            dr = wap.conv_desc(N, H, W, C, K, k, k, 1, pad, relu=relu)
            wap.wap_conv2d_fwd(dr, xd, wd, torch.from_numpy(bias).cuda() if relu else None, y, ws)
            torch.cuda.synchronize()
            want = np.maximum(ref + bias.astype(np.float64), 0.0) if relu else ref
            assert torch.isnan(y[-8:].float()).all() and gu.rel_err(gu.host_f64(y[:-8]).reshape(want.shape), want) <= gu.TOL_BF16_OUT
    if dx is None:
        return
    assert _flat(wap, d, wap.WAP_PASS_BWD_DATA) == dx
    need = wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_DATA)
    ref = orc.conv2d_bwd_data(g64, w64, (N, H, W, C), (1, 1), (pad, pad))
    out = torch.full((N * H * W * C + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = gu.workspace(need)
    wap.wap_conv2d_bwd_data(d, gd, wd, out, ws)
    torch.cuda.synchronize()
    assert torch.isnan(out[-8:].float()).all() and gu.rel_err(gu.host_f64(out[:-8]).reshape(ref.shape), ref) <= gu.TOL_BF16_OUT
    wap.wap_conv2d_bwd_data_relu(d, gd, wd, xd, out, ws)
    torch.cuda.synchronize()
    assert gu.rel_err(gu.host_f64(out[:-8]).reshape(ref.shape), np.where(x64 > 0, ref, 0.0)) <= gu.TOL_BF16_OUT
    if d.P % 2 or d.Q % 2:
        return
    am = si.rng(985, K).integers(0, 4, (N, d.P // 2, d.Q // 2, K)).astype(np.uint8)
    gpb = si.normal_bf16(si.rng(986, K), am.shape)
    gp = orc.bf16_bits_to_f64(gpb)
    full = np.zeros((N, d.P, d.Q, K))
    for i in range(4):
        full[:, i // 2::2, i % 2::2] = np.where(am == i, gp, 0.0)
    dy = torch.empty((N, d.P, d.Q, K), dtype=torch.bfloat16, device="cuda")
    wap.wap_conv2d_bwd_data_pool2x2(d, gu.dev_bf16(gpb), torch.from_numpy(am).cuda(), wd, None, out, dy, gu.workspace(need))
    torch.cuda.synchronize()
    ref = orc.conv2d_bwd_data(full, w64, (N, H, W, C), (1, 1), (pad, pad))
    assert gu.rel_err(gu.host_f64(out[:-8]).reshape(ref.shape), ref) <= gu.TOL_BF16_OUT
