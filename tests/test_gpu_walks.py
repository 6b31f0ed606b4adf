"""GPU: conversions and max-pools of odd channel counts that have more items than 4096 work-groups have threads."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4 << 20, (4 << 20) + 7, (60 << 20) - 5, (60 << 20) + 3])
def test_cast(n):
    import paper_1811_01532_amd as wap
    print(f"[case] cast {n}", flush=True)
    x = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    y = torch.full((n + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
    wap.wap_cast_f32_bf16(n, x, y)
    torch.cuda.synchronize()
    assert torch.equal(y[:n], x.to(torch.bfloat16)) and (y[n:] == 7.0).all()


@pytest.mark.parametrize("N,H,C,win,st", [(30, 61, 45, 2, 2), (9, 64, 81, 2, 1), (19, 70, 51, 3, 2), (25, 90, 21, 3, 3)])
def test_pools(N, H, C, win, st):
    """More than 2^20 items in one call, and the same images in calls of one, whose items are fewer: equal bits."""
    import paper_1811_01532_amd as wap
    print(f"[case] pool {N} x {H} x {H} x {C} window {win} stride {st}", flush=True)
    P = (H - win) // st + 1
    g = torch.Generator(device="cuda").manual_seed(N)
    x, dy = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((N, H, H, C), (N, P, P, C)))

    def pool(x, dy):
        n, y, dx = x.shape[0], torch.zeros_like(dy), torch.full_like(x, 7.0)
        am = torch.full(dy.shape, 255, dtype=torch.uint8, device="cuda")
        wap.wap_maxpool_fwd(n, H, H, C, win, st, x, y, am)
        wap.wap_maxpool_bwd(n, H, H, C, win, st, dy, am, y, dx)
        return y, am, dx

    whole, single = pool(x, dy), [pool(x[n:n + 1].clone(), dy[n:n + 1].clone()) for n in range(N)]
    torch.cuda.synchronize()
    assert all(torch.equal(a, torch.cat(b)) for a, b in zip(whole, zip(*single)))
    win_max = torch.stack([x[:, r:r + (P - 1) * st + 1:st, s:s + (P - 1) * st + 1:st] for r in range(win) for s in range(win)]).amax(0)
    assert torch.equal(whole[0], win_max)
