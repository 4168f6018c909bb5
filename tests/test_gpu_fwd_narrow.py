"""eq. (1) of arxiv 2411.01238 (Section 3.1) on 128 x 128 output tiles, which serve outputs too small to fill the chip with
128 x 256 ones: the same products in the same order, so the same bits as a call whose output is wide enough for the other form."""
import pytest
import torch

from oracle import sdrop_oracle as orc
from paper_2411_01238_amd import sdrop
from paper_2411_01238_amd.workloads import make_custom
from _util import f64, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,out", [("bf16", None), ("f16", torch.float32)])
@pytest.mark.parametrize("nk", [False, True])
@pytest.mark.parametrize("M,K,N,BK,p", [
    (128, 128, 8, 128, 0.0),            # one slice pair, eight columns
    (256, 192, 120, 64, 0.5),           # ragged, narrower than the tile
    (128, 256, 128, 128, 0.5),          # exactly one tile
    (384, 256, 136, 128, 0.3),          # a second tile column of eight
    (256, 512, 256, 64, 0.9),           # rows with nothing kept among them
    (4096, 256, 1024, 128, 0.5),        # the most tiles it is used for
    (129 * 128, 128, 128, 128, 0.5),    # a grid too tall for the seeded form
])
def test_same_bits_as_wide_tiles(M, K, N, BK, p, nk, dtype, out):
    print("fwd_narrow", M, K, N, BK, p, nk, dtype, flush=True)
    X, W, _ = make_custom(M, K, N, dtype, seed=5)
    Xg, Wg = X.cuda(), W.cuda()
    od = out or X.dtype
    Wl = Wg.t().contiguous() if nk else Wg
    y, m = sdrop.sdrop_fwd_seeded(Xg, Wl, 128, BK, p, 4, 2, out_dtype=od, w_layout=sdrop.W_NK if nk else sdrop.W_KN)
    y_obj = sdrop.sdrop_fwd_ex(Xg, Wl, m, out_dtype=od, w_layout=sdrop.W_NK if nk else sdrop.W_KN)
    # the same rows of X with the weight's columns repeated until the output fills the chip with wide tiles
    reps = -(-(256 * 128 * 256) // (M * N)) + 1
    wide = sdrop.sdrop_fwd(Xg, torch.cat([Wg] * reps, 1).contiguous(), m, out_dtype=od)
    torch.cuda.synchronize()
    assert torch.equal(y, wide[:, :N]) and torch.equal(y_obj, y)
    if M * K * N <= 1 << 25 and od == torch.float32:
        keep = orc.mask(M // 128, K // BK, p, 4, 2)
        assert_close(f64(y), orc.fwd(f64(X), f64(W), keep, 128, BK, p), "narrow forward")
