"""GPU parity of the fully-connected forward stream with two and four blocks of 16 batch rows: rows around the blocks, whole and partial
vectors, features that no work-group divides, divided and undivided reductions, with and without a workspace; an infinite weight among the
elements that a row's last vector shares with its neighbour reaches its own feature alone."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# rows, inputs, outputs, and the stream's template arguments in the queried workspace (None: on the other side of the line, the generic kernel)
CASES = [(17, 64, 16, (True, 2)), (31, 512, 1000, (True, 2)), (32, 4096, 1000, (True, 2)), (33, 4096, 500, (True, 4)), (48, 1000, 333, (True, 4)),
         (63, 67, 41, (False, 4)), (64, 9216, 512, None), (64, 515, 4096, (False, 4)), (20, 1024, 8192, None), (40, 22000, 80, (True, 4)), (64, 8, 9, (True, 4)),
         (18, 9, 24, (False, 2)), (20, 27, 40, (False, 2)), (25, 13, 700, (False, 2)), (29, 4099, 515, (False, 2)), (30, 5121, 200, (False, 2)),
         (32, 1003, 1000, (False, 2)), (17, 11003, 90, (False, 2)), (64, 2107, 90, (False, 4)), (63, 1344, 500, None), (33, 2112, 512, None),
         (43, 7011, 512, (False, 4)), (45, 2014, 500, (False, 4)), (38, 2013, 500, None), (61, 325, 174, (False, 4)), (32, 4837, 1200, None)]
# rows that the generic kernel takes, in the workspace that is enough for more rows, bytes
SHORT = [(63, 1344, 500, 0), (58, 1088, 572, 0), (33, 2112, 512, 409600), (61, 1152, 500, 0), (49, 1933, 4096, 0)]


@pytest.mark.parametrize("B,n_in,n_out,nws", [c[:3] + (None,) for c in CASES] + SHORT)
def test_forward_stream_of_several_row_blocks(orc, B, n_in, n_out, nws):
    """nws: bytes of workspace, None: what the query says.  (Which kernel each case runs is asserted without a GPU, in test_plans.py.)"""
    import paper_1811_01532_amd as wap
    print(f"[case] fc fwd {B} x {n_in} -> {n_out}", flush=True)
    x = orc.bf16_bits_to_f64(si.normal_bf16(si.rng(960, B + n_in), (B, n_in)))
    x[x == 0] = 1.0
    W = orc.bf16_bits_to_f64(si.he_weight_bf16(si.rng(961, n_in + n_out), (n_out, n_in)))
    bias = si.rng(962, n_out).standard_normal(n_out).astype(np.float32)
    for inf in (False, True):
        if inf:
            for i, col in enumerate(sorted({0, n_in - 8, n_in - 1 - n_in % 8, n_in - 1})):
                W[i, col] = np.inf if i % 2 else -np.inf
        xd, Wd = (gu.dev_bf16(si.f32_to_bf16_bits(t.astype(np.float32))) for t in (x, W))
        for relu in (False, True):
            d = wap.fc_desc(B, n_in, n_out, relu=relu)
            nbytes = wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD) if nws is None else nws
            ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
            ref = orc.fc_fwd(x, W, bias=bias.astype(np.float64), relu=relu)
            y = torch.full((B * n_out + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
            wap.wap_fc_fwd(d, xd, Wd, torch.from_numpy(bias).cuda(), y, ws)
            torch.cuda.synchronize()
            got, at = gu.host_f64(y[:B * n_out]).reshape(B, n_out), np.isinf(ref)
            assert torch.isnan(y[B * n_out:]).all() and np.array_equal(got[at], ref[at]) and (at.any() == inf)
            assert gu.rel_err(np.where(at, 0.0, got), np.where(at, 0.0, ref)) <= gu.TOL_BF16_OUT
