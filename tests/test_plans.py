"""CPU-only checks of what a plan promises its caller: which calls need no scratch tensor, which need no workspace."""
import pytest


@pytest.fixture(scope="module")
def wap():
    import paper_1811_01532_amd as w
    w.lib()
    return w


@pytest.mark.parametrize("N,H,W,C,K,pad", [(12, 12, 14, 256, 32, 2), (28, 18, 18, 64, 32, 2), (28, 18, 18, 64, 64, 2), (4, 24, 24, 256, 64, 2),
                                           (28, 24, 26, 64, 64, 2), (20, 24, 26, 128, 64, 2), (1, 48, 48, 256, 32, 2), (70, 20, 20, 64, 64, 0)])
def test_pooled_5x5_data_gradients_need_no_scratch_tensor(wap, N, H, W, C, K, pad):
    """Even 5x5 maps on tiles of whole patches: the gradient of the pooled output is routed while the patch is staged."""
    assert wap.wap_conv2d_bwd_pool2x2_fused(wap.conv_desc(N, H, W, C, K, 5, 5, 1, pad), wap.WAP_PASS_BWD_DATA)
