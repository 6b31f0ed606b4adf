"""GPU parity at the sizes where a kernel's layout or a dispatch rule changes: edges of tiles, remainders, the smallest and
largest shapes of a branch, each against the fp64 oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# rows around the limit of one row chunk (16 per thread of 1024: 1024 with 16 vectors side by side, 8192 with two, 256
# with 64 scalars) and of the small work-group (two rows per thread of 256), 16- / 8- / 2-byte vectors, column blocks
# with a ragged end
@pytest.mark.parametrize("rows,cols", [(1024, 128), (1025, 128), (8192, 16), (8193, 16), (32, 500), (33, 500), (3, 4),
                                       (256, 125), (257, 125), (70, 3), (100, 4096), (2000, 136)])
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
