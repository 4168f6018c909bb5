"""A layer's own bias in the forward kernel's epilogue (sdrop_fwd_seeded_bias) and its gradient (sdrop_col_sum): arxiv
2411.01238, eq. (1) with the bias of the linear layer behind the dropout, against float64 and against the plain calls."""
import numpy as np
import pytest
import torch

from oracle import sdrop_oracle as orc
from paper_2411_01238_amd import sdrop
from paper_2411_01238_amd.autograd import SparseDropLinear, sparsedrop_matmul
from paper_2411_01238_amd.workloads import make_custom
from _util import f64

pytestmark = pytest.mark.gpu

# unit spacing of the type relative to a value at the bottom of its binade: one rounding moves a value by at most half of it
EPS = {"bf16": 2.0 ** -7, "f16": 2.0 ** -10}


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N,BM,BK,nk", [
    (128, 128, 8, 128, 128, False),          # one tile, eight valid columns
    (256, 256, 256, 64, 64, False),
    (256, 384, 264, 128, 64, False),         # the last tile column eight wide
    (192, 256, 1000, 64, 128, False),
    (256, 256, 512, 128, 128, True),         # the weight as [N,K], in place
    (128, 256, 256, 64, 64, True),
    (256, 256, 72, 128, 128, True),          # ... through a transposed copy
    (129 * 64, 128, 256, 64, 64, False),     # a grid too tall for the seeded form: mask, then the product
    (129 * 64, 128, 520, 64, 64, False),
    (129 * 128, 128, 256, 128, 128, True),
    # 128 x 256 tiles with the mask drawn in the launch: whole, ragged, [N,K], more tiles than CUs (a workgroup reads its
    # bias values anew for each), and without the draw
    (8192, 256, 1024, 128, 128, False),
    (8192, 128, 1000, 128, 128, False),
    (8192, 256, 1536, 128, 128, True),
    (16384, 128, 1032, 128, 64, False),
    (129 * 128, 128, 512, 128, 128, False),
    (129 * 128, 128, 264, 128, 128, False),
])
def test_forward_with_bias(M, K, N, BM, BK, nk, dtype):
    p = 0.4
    print("bias case", M, K, N, BM, BK, nk, dtype, flush=True)
    X, W, _ = make_custom(M, K, N, dtype, seed=7)
    g = torch.Generator().manual_seed(1)
    b = torch.randn(N, generator=g).to(X.dtype)
    Wg = (W.t().contiguous() if nk else W).cuda()
    lay = sdrop.W_NK if nk else sdrop.W_KN
    guard = torch.full((M + 2, N), 7.0, dtype=X.dtype, device="cuda")
    y, m = sdrop.sdrop_fwd_seeded(X.cuda(), Wg, BM, BK, p, 3, 1, w_layout=lay, bias=b.cuda(), out=guard[1:M + 1])
    y0, m0 = sdrop.sdrop_fwd_seeded(X.cuda(), Wg, BM, BK, p, 3, 1, w_layout=lay)
    torch.cuda.synchronize()
    assert bool((guard[0] == 7).all()) and bool((guard[M + 1] == 7).all())
    assert torch.equal(m.bits(), m0.bits())
    assert torch.equal(y, y0 + b.cuda())        # the plain call's output with the bias added to it
    keep = orc.mask(M // BM, K // BK, p, 3, 1)
    if M <= 256:
        # two roundings: half a unit of the product and half a unit of the sum, plus the fp32 accumulation
        prod = orc.fwd(f64(X), f64(W), keep, BM, BK, p)
        ref = prod + f64(b)
        bound = 0.5 * EPS[dtype] * (np.abs(prod) + (1 + EPS[dtype]) * np.abs(ref)) + 2e-5 * np.max(np.abs(ref))
        assert np.all(np.abs(f64(y) - ref) <= bound)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("M,N,ld", [(1, 8, 8), (7, 64, 64), (64, 72, 72), (33, 128, 136), (300, 136, 136), (4096, 72, 72),
                                    (1000, 1000, 1024), (2048, 264, 264), (16384, 3072, 3072)])
def test_column_sums(M, N, ld, dtype):
    print("col_sum case", M, N, ld, dtype, flush=True)
    g = torch.Generator().manual_seed(M + N)
    d = torch.randn(M, N, generator=g).to(dtype)
    wide = torch.full((M, ld), float("nan"), dtype=dtype, device="cuda")
    wide[:, :N] = d.cuda()
    got = sdrop.sdrop_col_sum(wide[:, :N])
    ref = d.to(torch.float64).sum(0)
    # one rounding to the output type, plus fp32 sums in chains of at most M / 256 + 64 additions (rows of a thread, row
    # groups of a workgroup, parts), each off by 2^-24 of a partial sum that the sum of the magnitudes bounds
    eps = 0.5 * EPS["bf16" if dtype == torch.bfloat16 else "f16"]
    bound = eps * ref.abs() + 2.0 ** -24 * (M / 256 + 64) * d.to(torch.float64).abs().sum(0)
    assert bool(((got.cpu().to(torch.float64) - ref).abs() <= bound * 1.01).all())
    assert torch.equal(got, sdrop.sdrop_col_sum(wide[:, :N]))


def test_infinities_and_nan_go_where_they_belong():
    """Non-finite values of a bias and of dY reach their own columns, and only those."""
    print("bias non-finite", flush=True)
    inf, nan = float("inf"), float("nan")
    M, K, N = 256, 256, 264
    X, W, _ = make_custom(M, K, N, "bf16", seed=4)
    b = torch.zeros(N, dtype=torch.bfloat16)
    b[3], b[64], b[263] = inf, -inf, nan
    for B in (64, 128):
        y, _ = sdrop.sdrop_fwd_seeded(X.cuda(), W.cuda(), B, B, 0.3, 3, 1, bias=b.cuda())
        y0, _ = sdrop.sdrop_fwd_seeded(X.cuda(), W.cuda(), B, B, 0.3, 3, 1)
        assert torch.equal(y.isnan().cpu(), b.isnan().expand(M, N)) and torch.equal(y.nan_to_num(), (y0 + b.cuda()).nan_to_num())
    for rows in (7, 1000):
        d = torch.randn(rows, N, dtype=torch.float32).to(torch.bfloat16)
        d[rows - 1, 0], d[2, 63] = inf, -inf
        d[1, 127], d[5, 127] = inf, -inf           # of both signs: no number
        d[4, 263] = nan
        got, ref = sdrop.sdrop_col_sum(d.cuda()).cpu().double(), d.double().sum(0)
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf())
        assert torch.equal(got[got.isinf()], ref[ref.isinf()])


@pytest.mark.parametrize("bias_dtype", [torch.bfloat16, torch.float32])
def test_layer_gradients_and_the_forms_that_stay_torch(bias_dtype):
    torch.manual_seed(0)
    layer = SparseDropLinear(256, 72, p=0.5, BM=64, BK=64, bias=True, seed=2)
    layer.bias.data = torch.randn(72, device="cuda").to(bias_dtype)         # fp32: added as a torch operation, the output is fp32
    x = torch.randn(128, 256, device="cuda", dtype=torch.bfloat16, requires_grad=True)
    y = layer(x)
    assert y.dtype == bias_dtype
    dy = torch.randn(128, 72, device="cuda", dtype=y.dtype)
    dx, dw, db = torch.autograd.grad(y, [x, layer.weight, layer.bias], dy)
    assert db.dtype == bias_dtype
    ref = f64(dy).sum(0)
    # an fp32 sum of 128 values errs by less than 128 * 2^-24 of the magnitudes' sum; a bf16 one is rounded as well
    eps = 0.5 * EPS["bf16"] if bias_dtype == torch.bfloat16 else 0.0
    assert np.all(np.abs(f64(db) - ref) <= eps * np.abs(ref) + 128 * 2.0 ** -24 * np.abs(f64(dy)).sum(0))
    # the gradient of the bias is linear in dy and can be differentiated again
    dy.requires_grad_(True)
    layer.calls = 0
    (db2,) = torch.autograd.grad(layer(x), [layer.bias], dy, create_graph=True)
    (ddy,) = torch.autograd.grad(db2.float().sum(), [dy])
    assert bool((ddy == 1).all())


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N,B,layout,train", [
    (256, 256, 72, 64, "kn", True), (512, 256, 256, 128, "nk", True), (256, 256, 1000, 64, "kn", False), (256, 256, 72, 128, "nk", True),
])
def test_layer_with_a_bias_is_the_product_plus_the_bias(M, K, N, B, layout, train, dtype):
    """The layer's output and gradients are those of the product and an addition, whichever kernel adds the bias."""
    print("layer with bias", M, K, N, B, layout, train, dtype, flush=True)
    X, W, dY = make_custom(M, K, N, dtype, seed=11)
    dt = X.dtype
    layer = SparseDropLinear(K, N, p=0.3, BM=B, BK=B, bias=True, seed=5, dtype=dt, weight_layout=layout)
    g = torch.Generator().manual_seed(2)
    with torch.no_grad():
        layer.weight.copy_(W.t() if layout == "nk" else W)
        layer.bias.copy_(torch.randn(N, generator=g))
    layer.train(train)
    x = X.cuda().requires_grad_(True)
    dy = dY.cuda()
    y = layer(x)
    y0 = sparsedrop_matmul(x, layer.weight, 0.3 if train else 0.0, B, B, 5, 0, layout) + layer.bias
    assert torch.equal(y, y0)
    got = torch.autograd.grad(y, [x, layer.weight, layer.bias], dy)
    want = torch.autograd.grad(y0, [x, layer.weight], dy)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    ref = f64(dY).sum(0)
    assert np.all(np.abs(f64(got[2]) - ref) <= 0.5 * EPS[dtype] * np.abs(ref) + 1e-5 * np.abs(f64(dY)).sum(0))
    # a batch of sequences is the same matrix
    layer.calls = 0
    assert torch.equal(layer(X.cuda().view(2, M // 2, K)).view(M, N), y)
