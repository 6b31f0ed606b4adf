"""GPU parity of the fully-connected weight gradient as a stream of the weights: batch rows around the MFMA's 32, columns and rows
around a wavefront's blocks (16 rows, 64 and 128 columns), outputs of one row and of several blocks a wavefront, stored and applied
to the parameters, against the fp64 oracle and, bit for bit, against the update in a call of its own."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [(1, 4, 1), (3, 60, 15), (8, 128, 16), (16, 132, 17), (31, 520, 250), (32, 64, 48), (33, 4096, 333), (64, 124, 33), (65, 100, 40), (96, 192, 100),
         (97, 36, 20), (128, 1028, 66), (7, 2304, 1000)]


@pytest.mark.parametrize("B,n_in,n_out", CASES)
def test_weight_gradient_stream(orc, B, n_in, n_out):
    import paper_1811_01532_amd as wap
    assert wap.wap_conv2d_kernel_name(wap.conv_desc(B, 1, 1, n_in, n_out, 1, 1, 1, 0), wap.WAP_PASS_BWD_WEIGHT) == "fc_dw_kernel"
    print(f"[case] fc dW {B} x {n_in} -> {n_out}", flush=True)
    xb, gb = si.normal_bf16(si.rng(950, B + n_in), (B, n_in)), si.normal_bf16(si.rng(951, B + n_out), (B, n_out))
    xd, gd = gu.dev_bf16(xb), gu.dev_bf16(gb)
    d, n, lr = wap.fc_desc(B, n_in, n_out), n_in * n_out, 0.05
    dw = torch.full((n + 8,), float("nan"), device="cuda")
    wap.wap_fc_bwd(d, xd, None, gd, None, dw, None)
    w32 = torch.from_numpy(si.rng(952, n).standard_normal(n + 8).astype(np.float32)).cuda()
    w2, wb, wb2 = w32.clone(), torch.full((n + 8,), 7.0, dtype=torch.bfloat16, device="cuda"), torch.empty(n, dtype=torch.bfloat16, device="cuda")
    wap.wap_fc_bwd_weight_sgd(d, xd, gd, w32, wb, lr, None, None)
    wap.wap_sgd_update(n, w2, dw, lr, wb2)
    torch.cuda.synchronize()
    ref = orc.fc_bwd_weight(orc.bf16_bits_to_f64(gb), orc.bf16_bits_to_f64(xb))
    assert gu.rel_err(gu.host_f64(dw[:n]).reshape(n_out, n_in), ref) <= gu.TOL_F32_OUT
    assert torch.equal(w32, w2) and torch.equal(wb[:n].view(torch.int16), wb2.view(torch.int16))
    assert torch.isnan(dw[n:]).all() and (wb[n:] == 7.0).all()
