"""The products of a block's backward in pairs (sdrop_bwd_gated, sdrop_producer_bwd; arxiv 2411.01238, eq. (1)-(3) and Section
4.3's closing remark) bit for bit against the separate calls, which are held against the oracle elsewhere."""
import re

import pytest
import torch

from paper_2411_01238_amd import sdrop
from _util import kernel_names

pytestmark = pytest.mark.gpu


def _pair_forms(fn):
    """[(kernel, its tile widths), ...] of the paired kernels that one call launches."""
    forms = []
    for name in kernel_names(fn):
        k = re.search(r"(bwd_gated_kernel|fwd_dw_kernel)I", name)
        if k:
            widths = [int(v) for v in re.findall(r"Li(\d+)E", name[k.end():])]
            forms.append((k[1], widths[1:] if k[1] == "bwd_gated_kernel" else widths))      # (the gate's kernel: its tail first)
    return forms


# tiles: (width of dW's tiles, width of dH's), or None where the products run one after the other
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("gate_mode", [sdrop.GATE_RELU, sdrop.GATE_GELU_TANH, sdrop.GATE_GELU_ERF])
@pytest.mark.parametrize("M,K,N,BM,BK,p,tiles", [
    (128, 128, 256, 128, 128, 0.0, (256, 128)),         # one block
    (256, 384, 512, 128, 128, 0.5, (256, 128)),         # dW lists of one part, dX's reduction the longer one
    (512, 512, 256, 128, 128, 0.4, (128, 128)),         # dW on narrow tiles, one part
    (1024, 512, 256, 128, 128, 0.3, (128, 128)),        # ... its parts summed in the accumulators
    (1024, 512, 256, 128, 128, 1.0, (128, 128)),        # nothing kept
    (8192, 256, 512, 128, 128, 0.3, (256, 128)),        # dW cut into parts: fp32 planes and their sum
    (1024, 2048, 2048, 128, 128, 0.3, (256, 128)),      # more dX tiles and dW tiles than CUs
    (16384, 1024, 512, 128, 128, 0.1, (256, 256)),      # 256-wide forward tiles beside a dW in parts
    (2304, 4096, 2048, 128, 128, 0.5, (256, 256)),      # ... beside a whole one
    (12800, 128, 512, 128, 128, 0.1, None),             # long lists on narrow tiles
    (16384, 256, 256, 128, 128, 0.0, None),
    (256, 256, 264, 128, 128, 0.4, None),               # no whole tile columns
    (256, 256, 256, 64, 128, 0.4, None),                # other blocks
])
def test_bits_of_the_separate_calls(M, K, N, BM, BK, p, tiles, gate_mode, dtype):
    print("pair case", M, K, N, BM, BK, p, gate_mode, dtype, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def rand(*shape):
        return torch.randn(shape, generator=g, device="cuda").to(dtype)

    dY, W, X, gate = rand(M, N), rand(K, N), rand(M, K), rand(M, K)
    m = sdrop.sdrop_mask(M, K, BM, BK, p, 7)
    dz, dw = sdrop.sdrop_bwd_gated(dY, W, X, gate, gate_mode, m)
    dz0 = sdrop.sdrop_bwd_dx_ex(dY, W, m, relu_mask=gate, gate_mode=gate_mode)
    assert torch.equal(dz, dz0) and torch.equal(dw, sdrop.sdrop_bwd_dw(X, dY, m))
    dh, dw0 = sdrop.sdrop_producer_bwd(dz, W, dY, m)            # (W0 = W, H = dY: any [K, N0] and [M, N0])
    assert torch.equal(dh, sdrop.sdrop_fwd_ex(dz, W, m, scale_mode=sdrop.SCALE_ONE))
    assert torch.equal(dw0, sdrop.sdrop_bwd_dw_ex(dz, dY, m, scale_mode=sdrop.SCALE_ONE))
    # ... by the form this case is here for, not by the separate calls again
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        gated = _pair_forms(lambda: sdrop.sdrop_bwd_gated(dY, W, X, gate, gate_mode, m))
        producer = _pair_forms(lambda: sdrop.sdrop_producer_bwd(dz, W, dY, m))
        assert gated == ([] if tiles is None else [("bwd_gated_kernel", [tiles[0]])])
        assert producer == ([] if tiles is None else [("fwd_dw_kernel", [tiles[1], tiles[0]])])


def test_what_the_pairs_refuse():
    M, K, N = 256, 256, 256
    t = torch.zeros(M, K, device="cuda", dtype=torch.bfloat16)
    m = sdrop.sdrop_mask(M, K, 128, 128, 0.5, 1)
    with pytest.raises(ValueError):                             # rows of a wider matrix: the calls with leading dimensions
        sdrop.sdrop_bwd_gated(torch.zeros(M, N + 8, device="cuda", dtype=t.dtype)[:, :N], t, t, t, 0, m)
    with pytest.raises(sdrop.SdropError):
        sdrop.sdrop_bwd_gated(t, t, t, t, 9, m)
    with pytest.raises(ValueError):
        sdrop.sdrop_producer_bwd(t, t.half(), t, m)
