"""Operands that go to LDS through registers (arxiv 2411.01238, eq. (1)-(3) where N is no multiple of the tile or of the slice
of the reduction): chunks beyond the operand's end, which are fetched from the start of their row, reach no result."""
import pytest
import torch

from paper_2411_01238_amd import sdrop

pytestmark = pytest.mark.gpu


def _rand(shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(dtype)


@pytest.mark.parametrize("dtype,out", [(torch.bfloat16, None), (torch.float16, torch.float32)])
@pytest.mark.parametrize("M,K,N,BM,BK", [
    (256, 256, 264, 128, 128),      # eight columns in the last tile
    (128, 192, 72, 64, 64),         # one tile, less than half of it
    (512, 384, 504, 128, 64),       # all but eight columns of the last tile
])
def test_columns_beyond_n_reach_no_column_of_the_product(M, K, N, BM, BK, dtype, out):
    # the columns that stand in for those beyond N hold NaN and infinities: eq. (1) with an element-wise tail, eq. (3)
    print("ragged columns", M, K, N, BM, BK, dtype, out, flush=True)
    X, W, dY = _rand((M, K), dtype, 1), _rand((K, N), dtype, 2), _rand((M, N), dtype, 3)
    m = sdrop.sdrop_mask(M, K, BM, BK, 0.25, 5)
    bias = _rand((N,), torch.float32, 4)
    bad_w, bad_dy = W.clone(), dY.clone()
    bad_w[:, :8] = float("nan")
    bad_dy[:, :8] = float("inf")
    for act in (sdrop.ACT_GELU_ERF, sdrop.ACT_RELU):
        y = sdrop.sdrop_fwd_ex(X, W, m, act=act, bias=bias, out_dtype=out)
        bad = sdrop.sdrop_fwd_ex(X, bad_w, m, act=act, bias=bias, out_dtype=out)
        assert torch.equal(bad[:, 8:], y[:, 8:])
    dw = sdrop.sdrop_bwd_dw(X, dY, m, out_dtype=out)
    bad = sdrop.sdrop_bwd_dw(X, bad_dy, m, out_dtype=out)
    assert torch.equal(bad[:, 8:], dw[:, 8:])


@pytest.mark.parametrize("dtype,out", [(torch.bfloat16, None), (torch.float16, torch.float32)])
@pytest.mark.parametrize("M,K,N,BM,BK,p", [
    (256, 256, 72, 64, 64, 0.25),       # a slice and eight
    (192, 384, 120, 64, 128, 0.5),      # all but eight of the second slice
    (1024, 1024, 200, 128, 128, 0.1),   # 256-wide tiles, a workgroup each
    (512, 512, 8, 128, 128, 0.0),       # nothing but the ragged slice
    (4096, 2560, 72, 128, 128, 0.1),    # the persistent kernel's own ragged slice
])
def test_a_ragged_reduction_equals_one_padded_with_zeros(M, K, N, BM, BK, p, dtype, out):
    # eq. (2): zeros add nothing to an fp32 sum, so the bits are those of the padded product
    print("ragged reduction", M, K, N, BM, BK, p, dtype, out, flush=True)
    dY, W = _rand((M, N), dtype, 1), _rand((K, N), dtype, 2)
    m = sdrop.sdrop_mask(M, K, BM, BK, p, 5)
    whole = -(-N // 64) * 64
    dYp, Wp = torch.zeros(M, whole, dtype=dtype, device="cuda"), torch.zeros(K, whole, dtype=dtype, device="cuda")
    dYp[:, :N], Wp[:, :N] = dY, W
    assert torch.equal(sdrop.sdrop_bwd_dx(dY, W, m, out_dtype=out), sdrop.sdrop_bwd_dx(dYp, Wp, m, out_dtype=out))
    gate = _rand((M, K), dtype, 3)
    got = sdrop.sdrop_bwd_dx_ex(dY, W, m, relu_mask=gate, gate_mode=sdrop.GATE_GELU_ERF, out_dtype=out)
    assert torch.equal(got, sdrop.sdrop_bwd_dx_ex(dYp, Wp, m, relu_mask=gate, gate_mode=sdrop.GATE_GELU_ERF, out_dtype=out))
