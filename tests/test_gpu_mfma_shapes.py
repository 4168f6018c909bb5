"""The forms of a product that run on 16 x 16 x 32 matrix instructions against those on 32 x 32 x 16 ones: the same bits
(eq. (1)-(3) of arxiv 2411.01238; either form is held against the float64 oracle elsewhere)."""
import pytest
import torch

from paper_2411_01238_amd import sdrop
from paper_2411_01238_amd.workloads import make_custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K,N", [(128, 256), (192, 264), (1024, 512)])
def test_wide_and_narrow_forward_tiles(K, N, dtype):
    # 100 (200) 128 x 256 tiles: wide ones (16 x 16); the same rows eight blocks at a time: 128 x 128 tiles (32 x 32)
    M, B = 12800, 64 if K % 128 else 128
    X, W, _ = make_custom(M, K, N, dtype, seed=11)
    X, W = X.cuda(), W.cuda()
    y = sdrop.sdrop_fwd(X, W, sdrop.sdrop_mask(M, K, 128, B, 0.0, 0))
    m = sdrop.sdrop_mask(1024, K, 128, B, 0.0, 0)
    for r in range(0, 12288, 4096):
        assert torch.equal(sdrop.sdrop_fwd(X[r:r + 1024], W, m), y[r:r + 1024])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("width", [128, 256])
def test_dx_against_a_forward_product(width, dtype):
    # with nothing dropped dX = dY W^T is a forward product with the weight W^T: eq. 2's kernels (16 x 16) against eq. 1 on
    # 128 x 128 tiles (32 x 32)
    M, K, N = 1024, 512, 320
    _, W, dY = make_custom(M, K, N, dtype, seed=12)
    W, dY = W.cuda(), dY.cuda()
    m, mt = sdrop.sdrop_mask(M, K, 128, 128, 0.0, 0), sdrop.sdrop_mask(M, N, 128, 64, 0.0, 0)
    try:
        sdrop.set_tuning(sdrop.TUNE_DX_TILE_WIDTH, width)
        dx = sdrop.sdrop_bwd_dx(dY, W, m)
    finally:
        sdrop.set_tuning(sdrop.TUNE_DX_TILE_WIDTH, 0)
    assert torch.equal(dx, sdrop.sdrop_fwd(dY, W.t().contiguous(), mt))
