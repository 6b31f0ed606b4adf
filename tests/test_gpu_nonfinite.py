"""An infinity or a NaN in the image reaches the outputs whose window it lies in and no others: the 11x11 first layer, whose filter
is padded to 12x12 inside the kernel, by groups of 1, 2 and 4 output rows."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,K,pad", [(4, 31, 138, 64, 2), (4, 43, 140, 32, 0), (20, 107, 226, 64, 2), (110, 55, 136, 32, 2)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_first_layer_windows(N, H, W, K, pad, value):
    import paper_1811_01532_amd as wap
    print(f"[case] non-finite 11x11 {(N, H, W, K, pad, value)}", flush=True)
    g = torch.Generator().manual_seed(77)
    x = torch.randn(N, H, W, 3, generator=g).bfloat16().cuda()
    w = torch.randn(K, 11, 11, 3, generator=g).bfloat16().cuda()
    d = wap.conv_desc(N, H, W, 3, K, 11, 11, 4, pad)
    assert wap.wap_conv2d_kernel_name(d, wap.WAP_PASS_FWD).startswith("conv_c3_fwd_strided_kernel")
    y0, y1 = (torch.empty(N, d.P, d.Q, K, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    wap.wap_conv2d_fwd(d, x, w, None, y0, None)
    # one pixel an image, on every residue of the stride: below, above and beside windows
    touched = torch.zeros(N, d.P, d.Q, dtype=torch.bool)
    for n in range(N):
        h, v = (7 * n + 11 - pad) % H, (5 * n + 23 - pad) % W
        x[n, h, v, n % 3] = value
        for p in range(d.P):
            for q in range(d.Q):
                touched[n, p, q] = 0 <= h + pad - 4 * p < 11 and 0 <= v + pad - 4 * q < 11
    wap.wap_conv2d_fwd(d, x, w, None, y1, None)
    torch.cuda.synchronize()
    y0, y1 = y0.cpu(), y1.cpu()
    assert torch.equal(y1[~touched].view(torch.int16), y0[~touched].view(torch.int16))
    assert touched.any() and not torch.isfinite(y1[touched].float()).any()
