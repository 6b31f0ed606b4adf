"""GPU parity of the 3x3 first layer whose output rows are whole 32-pixel tiles: fewer tiles than wavefronts, one and several tiles each, a last round
that is cut short, both channel counts, with and without padding; an infinity in the image reaches its own windows only."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [(1, 64, 64, 64, 1), (4, 32, 32, 32, 1), (3, 50, 66, 64, 0), (2, 96, 160, 32, 1), (7, 224, 224, 64, 1), (9, 130, 130, 64, 0), (31, 96, 96, 32, 1)]


@pytest.mark.parametrize("N,H,W,K,pad", CASES)
def test_first_layer_on_rows_of_whole_tiles(orc, N, H, W, K, pad):
    import paper_1811_01532_amd as wap
    print(f"[case] first layer {(N, H, W, K, pad)}", flush=True)
    d = wap.conv_desc(N, H, W, 3, K, 3, 3, 1, pad)
    assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_FWD).startswith("conv_c3_fwd_rows") and wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_BWD_WEIGHT).startswith("wgrad_c3_rows")
    xb, wb = si.normal_bf16(si.rng(970, N + H), (N, H, W, 3)), si.he_weight_bf16(si.rng(971, K), (K, 3, 3, 3))
    gb = si.normal_bf16(si.rng(972, N + W), (N, d.P, d.Q, K))
    x64, w64, g64 = (orc.bf16_bits_to_f64(t) for t in (xb, wb, gb))
    xd, wd, gd = (gu.dev_bf16(t) for t in (xb, wb, gb))
    y = torch.full((N * d.P * d.Q * K + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((K * 27 + 8,), float("nan"), device="cuda")
    wap.wap_conv2d_fwd(d, xd, wd, None, y, gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_FWD)))
    ws = gu.workspace(wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT))
    wap.wap_conv2d_bwd_weight(d, xd, gd, dw, ws)
    again = torch.empty_like(dw)
    wap.wap_conv2d_bwd_weight(d, xd, gd, again, ws)
    torch.cuda.synchronize()
    assert torch.isnan(y[-8:].float()).all() and torch.isnan(dw[-8:]).all() and torch.equal(dw[:-8], again[:-8])
    assert gu.rel_err(gu.host_f64(y[:-8]).reshape(N, d.P, d.Q, K), orc.conv2d_fwd(x64, w64, (1, 1), (pad, pad))) <= gu.TOL_BF16_OUT
    assert gu.rel_err(gu.host_f64(dw[:-8]).reshape(K, 3, 3, 3), orc.conv2d_bwd_weight(x64, g64, (K, 3, 3, 3), (1, 1), (pad, pad))) <= gu.TOL_F32_OUT
    # an infinity at the image's last column: finite outputs wherever no window holds it
    xd.view(N, H, W, 3)[0, H // 2, W - 1, 1] = float("inf")
    wap.wap_conv2d_fwd(d, xd, wd, None, y, None)
    torch.cuda.synchronize()
    bad = (~torch.isfinite(y[:-8].float())).view(N, d.P, d.Q, K).any(dim=3)
    at = bad.nonzero()
    assert len(at) > 0 and (at[:, 0] == 0).all() and (at[:, 1] >= H // 2 - 2 + pad).all() and (at[:, 1] <= H // 2 + pad).all() and (at[:, 2] >= W - 3 + pad).all()
