"""The forward without a mask (sdrop_fwd_dense): eq. (1) of arxiv 2411.01238 with nothing dropped, as a layer in inference
calls it, bit for bit against the seeded call with p = 0, which is held against the float64 oracle elsewhere."""
import pytest
import torch

from paper_2411_01238_amd import sdrop
from paper_2411_01238_amd.autograd import SparseDropLinear
from paper_2411_01238_amd.workloads import make_custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N,BM,BK,nk,bias", [
    (128, 64, 8, 64, 64, False, True),              # one tile of two block rows, one slice, eight valid columns
    (256, 192, 264, 64, 64, False, False),          # an odd number of 64-wide blocks; a ragged second tile column
    (8192, 1024, 1000, 64, 64, False, True),        # 128 x 256 tiles, a ragged last column
    (16384, 128, 1032, 128, 128, False, False),     # more tiles than CUs
    (130 * 64, 128, 256, 64, 64, False, False),     # a grid that the seeded form does not draw itself
    (256, 4096 + 64, 256, 64, 64, False, True),     # more than 64 block columns
    (512, 256, 512, 128, 64, True, True),           # the weight as [N,K]: 128-wide tiles
    (16384, 128, 512, 64, 128, True, False),        # ... 256-wide ones
])
def test_bits_of_the_seeded_forward(M, K, N, BM, BK, nk, bias, dtype):
    print("dense case", M, K, N, BM, BK, nk, bias, dtype, flush=True)
    X, W, _ = make_custom(M, K, N, dtype, seed=5)
    X, W = X.cuda(), (W.t().contiguous() if nk else W).cuda()
    b = torch.randn(N, generator=torch.Generator().manual_seed(1)).to(X.dtype).cuda() if bias else None
    lay = sdrop.W_NK if nk else sdrop.W_KN
    y0, _ = sdrop.sdrop_fwd_seeded(X, W, BM, BK, 0.0, 3, 1, w_layout=lay, bias=b)
    y = sdrop.sdrop_fwd_dense(X, W, BM, BK, w_layout=lay, bias=b)
    torch.cuda.synchronize()
    assert torch.equal(y, y0)
    # rows of a wider matrix
    wide = torch.randn(M, K + 8, device="cuda").to(X.dtype)
    wide[:, :K] = X
    assert torch.equal(sdrop.sdrop_fwd_dense(wide[:, :K], W, BM, BK, w_layout=lay, bias=b), y0)


def test_shapes_without_a_kernel_take_the_masked_call():
    X, W, _ = make_custom(192, 128, 72, "bf16", seed=5)
    assert sdrop.sdrop_fwd_dense(X.cuda(), W.cuda(), 64, 64) is None               # 64-row blocks, an odd number of them
    X, W, _ = make_custom(256, 128, 72, "bf16", seed=5)
    assert sdrop.sdrop_fwd_dense(X.cuda(), W.t().contiguous().cuda(), 64, 64, w_layout=sdrop.W_NK) is None
    with pytest.raises(sdrop.SdropError):
        sdrop.sdrop_fwd_dense(X[:96].contiguous().cuda(), W.cuda(), 64, 64)        # the block must divide the shape, as ever


@pytest.mark.parametrize("M", [192, 256])
def test_layer_in_inference(M):
    layer = SparseDropLinear(128, 264, 0.5, 64, 64, bias=True, seed=1).eval()
    x = torch.randn(M, 128, device="cuda").to(torch.bfloat16)
    with_graph = layer(x)
    assert with_graph.requires_grad
    with torch.no_grad():
        y = layer(x)
    assert not y.requires_grad and torch.equal(y, with_graph)
    with torch.inference_mode():
        assert torch.equal(layer(x), y)
