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


@pytest.fixture
def routes(monkeypatch):
    """The forward calls that a layer makes, by name (both give the same bits, so the result does not tell)."""
    seen = []

    def watch(name):
        call = getattr(sdrop, name)

        def watched(*a, **kw):
            r = call(*a, **kw)
            seen.append(name if r is not None else name + " without a kernel")
            return r
        monkeypatch.setattr(sdrop, name, watched)

    watch("sdrop_fwd_dense")
    watch("sdrop_fwd_seeded")
    return seen


@pytest.mark.parametrize("M,N,nk,route", [
    (256, 264, False, "sdrop_fwd_dense"), (192, 264, False, "sdrop_fwd_seeded"),
    (256, 256, True, "sdrop_fwd_dense"), (256, 264, True, "sdrop_fwd_seeded"),
])
def test_layer_in_inference(M, N, nk, route, routes):
    layer = SparseDropLinear(128, N, 0.5, 64, 64, bias=True, seed=1, weight_layout="nk" if nk else "kn").eval()
    x = torch.randn(M, 128, device="cuda").to(torch.bfloat16)
    with_graph = layer(x)
    assert with_graph.requires_grad and routes == ["sdrop_fwd_seeded"]
    with torch.no_grad():
        y = layer(x)
    assert not y.requires_grad and torch.equal(y, with_graph)
    with torch.inference_mode():
        assert torch.equal(layer(x), y)
    assert routes[1:] == [route, route]


def test_a_training_layer_drops_blocks_without_a_graph_too(routes):
    layer = SparseDropLinear(128, 264, 0.5, 64, 64, bias=False, seed=1)
    x = torch.ones(256, 128, device="cuda", dtype=torch.bfloat16)
    with torch.no_grad():
        layer.weight.fill_(1.0)
        y = layer(x)
    assert routes == ["sdrop_fwd_seeded"]
    keep = sdrop.sdrop_mask(256, 128, 64, 64, 0.5, 1, 0).bits().cpu().flatten().tolist()
    kept = torch.tensor([bin(b & 3).count("1") for b in keep]).repeat_interleave(64)
    assert torch.equal(y.float().cpu(), (kept * 128.0)[:, None].expand(-1, 264)) and 0 < kept.sum() < 2 * 256
