"""GPU parity of the weights in MFMA fragment order: reductions that are no whole run of four steps, output channels that are no
block of 32, no group of four and odd (data gradient: eight rows turned around in registers, or element by element)."""
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,C,K,back", [(1, 40, 32, 32, 128, False), (2, 28, 28, 96, 128, False),
                                            (1, 90, 90, 131, 64, True), (1, 90, 90, 132, 64, True), (1, 90, 90, 200, 64, True)])
def test_weights_in_fragment_order(orc, N, H, W, C, K, back):
    import paper_1811_01532_amd as wap
    print(f"[case] weight order {(N, H, W, C, K, back)}", flush=True)
    wb = si.he_weight_bf16(si.rng(941, K + C), (K, 3, 3, C))
    ib = si.normal_bf16(si.rng(942, C), (N, H, W, K if back else C))
    d = wap.conv_desc(N, H, W, C, K, 3, 3, 1, 1)
    p = wap.WAP_PASS_BWD_DATA if back else wap.WAP_PASS_FWD
    assert wap.wap_conv2d_kernel_name(d, p).startswith("conv_patch_kernel" if back else "conv_tile2d_kernel")
    out = torch.empty((N, H, W, C if back else K), dtype=torch.bfloat16, device="cuda")
    ws = gu.workspace(wap.wap_conv2d_workspace_bytes(d, p))
    if back:
        wap.wap_conv2d_bwd_data(d, gu.dev_bf16(ib), gu.dev_bf16(wb), out, ws)
    else:
        wap.wap_conv2d_fwd(d, gu.dev_bf16(ib), gu.dev_bf16(wb), None, out, ws)
    torch.cuda.synchronize()
    i64, w64 = orc.bf16_bits_to_f64(ib), orc.bf16_bits_to_f64(wb)
    ref = orc.conv2d_bwd_data(i64, w64, (N, H, W, C), (1, 1), (1, 1)) if back else orc.conv2d_fwd(i64, w64, (1, 1), (1, 1))
    assert gu.rel_err(gu.host_f64(out), ref) <= gu.TOL_BF16_OUT
