"""GPU: updates and ReLU derivatives on either side of the size from which they pass the cache give the same bits, whole and in pieces."""
import pytest
import torch

from tests import gpu_util as gu
from tests.test_gpu_step import _setup

pytestmark = pytest.mark.gpu

CACHE = 268435456
LINE = CACHE // 10  # up to this many parameters (fp32, gradient, bf16 copy) fit the cache
GRID, WALK = 1 << 20, 3 << 19  # vectors from which on 4096 work-groups walk, and from which on a thread has one again
LINES = [int(CACHE / 7.4), int(CACHE / 5.95)]  # from these on they pass it, with and without a bf16 copy


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 1027, 4 * GRID + 3, 4 * WALK - 1, 4 * WALK + 5, LINE, LINE + 1, LINE + 6, LINES[0] - 2, LINES[0] + 3, LINES[1] - 2, LINES[1] + 7])
@pytest.mark.parametrize("copy", [True, False])
def test_update_whole_and_in_pieces(n, copy):
    import paper_1811_01532_amd as wap
    print(f"[case] sgd {n} {copy}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    w, dw = (torch.randn(n + 8, generator=g, device="cuda") for _ in range(2))
    want = torch.addcmul(w[:n].double(), dw[:n].double(), torch.tensor(-0.1, device="cuda").double()).float()  # fp64: at most a tie apart
    w2, wb, wb2 = w.clone(), *(torch.full((n + 8,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    wap.wap_sgd_update(n, w, dw, 0.1, wb if copy else None)
    piece = (n // 3 + 7) // 8 * 8 + 8
    for at in range(0, n, piece):
        m = min(piece, n - at)
        wap.wap_sgd_update(m, w2[at:at + m], dw[at:at + m], 0.1, wb2[at:at + m] if copy else None)
    torch.cuda.synchronize()
    assert torch.equal(w, w2) and torch.equal(wb.view(torch.int16), wb2.view(torch.int16))
    assert (w[:n] - want).abs().max() <= 2.0 ** -22 * want.abs().max()
    assert not copy or torch.equal(wb[:n], w[:n].to(torch.bfloat16))
    assert (wb[n:] == 7.0).all()


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 2047, 2049, 8 * GRID + 7, 8 * WALK - 3, 8 * WALK + 5, 268435456 // 6, 268435456 // 6 + 5, int(CACHE / 5.35) - 3, int(CACHE / 5.35) + 5, 268435456 // 3 + 3])
def test_relu_derivative(n, in_place):
    import paper_1811_01532_amd as wap
    print(f"[case] relu_bwd {n} {in_place}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    dy, y = (torch.randn(n + 8, generator=g, device="cuda").bfloat16() for _ in range(2))
    y[:n:5] = 0.0
    dx = dy.clone() if in_place else torch.full_like(dy, 7.0)
    tail = dx[n:].clone()
    wap.wap_relu_bwd(dx if in_place else dy, y, dx, n)
    torch.cuda.synchronize()
    assert torch.equal(dx[:n].view(torch.int16), torch.where(y[:n] > 0, dy[:n], torch.zeros_like(dy[:n])).view(torch.int16))
    assert torch.equal(dx[n:], tail)


@pytest.mark.parametrize("B,n_in,n_out", [(5, 11008, 4096), (70, 11008, 4096), (130, 11008, 4096)])  # 45 M parameters, 6 bytes each
def test_fused_update_past_the_cache(B, n_in, n_out):
    import paper_1811_01532_amd as wap
    print(f"[case] fc dW + update {B} x {n_in} -> {n_out}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B)
    x, g = torch.randn(B, n_in, generator=gen, device="cuda").bfloat16(), torch.randn(B, n_out, generator=gen, device="cuda").bfloat16()
    n, d = n_in * n_out, wap.fc_desc(B, n_in, n_out)
    nws = wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_BWD_WEIGHT)
    ws = torch.empty(nws + 256, dtype=torch.uint8, device="cuda") if nws else None
    w32 = torch.randn(n, generator=gen, device="cuda")
    w2, dw = w32.clone(), torch.empty(n, device="cuda")
    wb, wb2 = (torch.empty(n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    assert wap.wap_fc_bwd_weight_sgd_fused(d)
    wap.wap_fc_bwd_weight_sgd(d, x, g, w32, wb, 0.05, None, ws)
    wap.wap_fc_bwd(d, x, None, g, None, dw, ws)
    for at in range(0, n, n // 8):
        wap.wap_sgd_update(n // 8, w2[at:at + n // 8], dw[at:at + n // 8], 0.05, wb2[at:at + n // 8])
    torch.cuda.synchronize()
    assert torch.equal(w32, w2) and torch.equal(wb.view(torch.int16), wb2.view(torch.int16))


# networks of more than 26.8 M parameters, whose stored gradients pass the cache: rows that stream, and rows that the tiles take
STEPS = [("alexnet", 33, 99), ("alexnet", 70, 99), ("vgg16", 129, 32), ("vgg16", 22, 32)]


@pytest.mark.parametrize("net,B,image", STEPS)
def test_stored_fully_connected_gradients(net, B, image):
    """Each layer's stored weight gradient against the fp64 product of the very operands that the plan keeps, with and without a kept
    copy of every intermediate."""
    import paper_1811_01532_amd as wap
    print(f"[case] stored gradients {net} B={B} image={image}", flush=True)
    plan, ar, shapes, fcs, *_ = _setup(net, B, image, wap.WAP_STEP_KEEP_GRADS, 560)
    plan.run(ar.buf)
    torch.cuda.synchronize()
    x = shapes[-1]["name"] + (".pool.y" if shapes[-1]["pool"] else ".y")
    plan2, ar2, *_ = _setup(net, B, image, wap.WAP_STEP_STORE_GRADS, 560)
    plan2.run(ar2.buf)
    torch.cuda.synchronize()
    for name, n_in, n_out, relu in fcs:
        g = ar.bf16(("gm." if relu else "g.") + name + ".y", (B, n_out)).double()
        ref = g.t().contiguous() @ ar.bf16(x, (B, n_in)).double()
        for a in (ar, ar2):
            e = (a.f32(name + ".dw", (n_out, n_in)).double() - ref).abs().max() / ref.abs().max()
            assert ref.abs().max() > 0 and e <= gu.TOL_F32_OUT, (name, float(e))
        x = name + ".y"
