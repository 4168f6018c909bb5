"""The pre-activation that sdrop_producer allocates itself (arxiv 2411.01238, Section 4.3's closing remark): zero in every
dropped block, and the caller's own tensor, whose dropped blocks are left alone, elsewhere."""
import pytest
import torch

from paper_2411_01238_amd import sdrop

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N0,BM,BK,p,out", [
    (256, 384, 256, 128, 128, 0.5, None),        # a workgroup per block position
    (4096, 2560, 128, 128, 128, 0.4, None),      # more positions than CUs
    (256, 256, 200, 128, 128, 0.5, None),        # a ragged reduction
    (256, 256, 128, 64, 64, 0.5, None),          # 64-row blocks, a workgroup per tile
    (128, 512, 72, 64, 128, 0.5, None),          # ... with a ragged reduction
    (512, 512, 128, 128, 64, 0.5, torch.float32),
    (256, 256, 128, 128, 128, 1.0, None),        # nothing kept
])
def test_dropped_blocks_are_zero(M, K, N0, BM, BK, p, out):
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    H = torch.randn(M, N0, generator=g, device="cuda").to(torch.bfloat16)
    W0 = torch.randn(K, N0, generator=g, device="cuda").to(torch.bfloat16)
    b0 = torch.randn(K, generator=g, device="cuda")
    m = sdrop.sdrop_mask(M, K, BM, BK, p, 5)
    z0 = torch.zeros(M, K, dtype=out or H.dtype, device="cuda")
    x0, _ = sdrop.sdrop_producer(H, W0, b0, m, act=sdrop.ACT_GELU_ERF, out_dtype=out, preact=z0)
    # (memory that is likely to be handed out again holds NaN)
    for _ in range(4):
        torch.full_like(z0, float("nan"))
    x, z = sdrop.sdrop_producer(H, W0, b0, m, act=sdrop.ACT_GELU_ERF, out_dtype=out, preact=True)
    assert torch.equal(x, x0) and torch.equal(z, z0)
    own = torch.full_like(z0, 7.0)
    sdrop.sdrop_producer(H, W0, b0, m, act=sdrop.ACT_GELU_ERF, out_dtype=out, preact=own)
    keep = torch.from_numpy(((m.bits().cpu().numpy().view("uint64")[:, :, None] >> torch.arange(64).numpy().astype("uint64")) & 1)
                            .reshape(M // BM, -1)[:, :K // BK].astype("uint8")).cuda().bool()
    keep = keep.repeat_interleave(BM, 0).repeat_interleave(BK, 1)
    assert torch.equal(own, torch.where(keep, z0, torch.full_like(z0, 7.0)))
