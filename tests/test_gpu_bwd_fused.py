"""sdrop_bwd: eq. (2) and eq. (3) of arxiv 2411.01238 (Section 3.1) in one call, and in one launch
where the shapes allow it.  Against the float64 oracle through the C ABI, and bit for bit against
the two separate entry points, with the single launch switched on and off."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import sdrop_oracle as orc
from paper_2411_01238_amd import sdrop
from paper_2411_01238_amd.workloads import make_custom
from _util import f64, assert_close, assert_bf16_rounding_of

pytestmark = pytest.mark.gpu

CASES = [
    # M, K, N, BM, BK, dtype, p, seed, dX kernel forced persistent
    (1024, 512, 512, 128, 128, "bf16", 0.5, 1, False),    # one launch: one kept block per dX tile, 8 dW tiles
    (1536, 256, 512, 128, 128, "f16", 0.3, 2, False),     # one launch; dW on 128 x 128 tiles, its parts summed in the accumulators
    (2048, 256, 512, 128, 128, "f16", 0.3, 12, False),    # one launch; the dW part writes split fp32 planes, a summing pass follows
    (2560, 2560, 256, 128, 128, "bf16", 0.1, 3, True),    # one launch: dX tiles of two kept blocks, persistent form
    (2560, 2560, 256, 128, 128, "f16", 0.1, 13, False),   # one launch: dX tiles of two kept blocks, a workgroup per tile
    (1536, 1536, 512, 128, 128, "bf16", 0.0, 14, False),  # nothing dropped, one kept block per dX tile, dW summed in the accumulators
    (2560, 2560, 512, 128, 128, "bf16", 0.0, 15, False),  # nothing dropped, dX tiles of two kept blocks and a split dW
    (4096, 1024, 256, 128, 128, "f16", 0.7, 4, False),    # one launch: more dX workgroups than kept blocks
    (512, 768, 328, 128, 128, "bf16", 0.3, 5, False),     # ragged N: two launches
    (384, 512, 256, 64, 64, "f16", 0.5, 6, False),        # 64 x 64 blocks, short kept lists: one launch, both a workgroup per tile
    (2048, 512, 256, 64, 64, "bf16", 0.3, 16, False),     # the same with dW split into parts and summed
    (4096, 256, 256, 64, 64, "bf16", 0.0, 17, False),     # 64 x 64 blocks, long kept lists (persistent dW): two launches
    (384, 512, 328, 64, 64, "f16", 0.5, 18, False),       # 64 x 64 blocks, ragged N: two launches
    (512, 512, 256, 128, 64, "bf16", 0.4, 7, False),      # 128 x 64 blocks: two launches
    (128, 128, 256, 128, 128, "bf16", 0.0, 8, False),     # a single block
]


@pytest.mark.parametrize("M,K,N,BM,BK,dtype,p,seed,force", CASES)
def test_both_gradients_in_one_call(M, K, N, BM, BK, dtype, p, seed, force):
    print("bwd fused", M, K, N, BM, BK, dtype, p, seed, force, flush=True)
    X, W, dY = make_custom(M, K, N, dtype, seed=seed)
    m = sdrop.sdrop_mask(M, K, BM, BK, p, seed, 0)
    keep = orc.mask(M // BM, K // BK, p, seed, 0)
    Xg, Wg, dYg = X.cuda(), W.cuda(), dY.cuda()
    ref_dx = orc.bwd_dx(f64(dY), f64(W), keep, BM, BK, p)
    ref_dw = orc.bwd_dw(f64(X), f64(dY), keep, BM, BK, p)
    if force:
        sdrop.set_tuning(sdrop.TUNE_DX_PERSISTENT_GROUPS_PER_CU, 0)
    try:
        for out_dtype in (torch.float32, None):
            sep_dx = sdrop.sdrop_bwd_dx(dYg, Wg, m, out_dtype=out_dtype)
            sep_dw = sdrop.sdrop_bwd_dw(Xg, dYg, m, out_dtype=out_dtype)
            for fused in (1, 0):
                sdrop.set_tuning(sdrop.TUNE_BWD_FUSED, fused)
                dx, dw = sdrop.sdrop_bwd(dYg, Wg, Xg, m, out_dtype=out_dtype)
                torch.cuda.synchronize()
                tag = "bwd(%d,%d,%d,%dx%d,%s) fused=%d out=%s" % (M, K, N, BM, BK, dtype, fused, out_dtype)
                assert torch.equal(dx, sep_dx), tag + ": dX differs from sdrop_bwd_dx"
                assert torch.equal(dw, sep_dw), tag + ": dW differs from sdrop_bwd_dw"
                if out_dtype == torch.float32 or X.dtype == torch.float16:
                    assert_close(f64(dx), ref_dx, tag + " dX")
                    assert_close(f64(dw), ref_dw, tag + " dW")
                else:
                    assert_bf16_rounding_of(f64(dx), ref_dx, tag + " dX")
                    assert_bf16_rounding_of(f64(dw), ref_dw, tag + " dW")
    finally:
        sdrop.set_tuning(sdrop.TUNE_BWD_FUSED, 1)
        sdrop.set_tuning(sdrop.TUNE_DX_PERSISTENT_GROUPS_PER_CU, sdrop.DX_PERSISTENT_GROUPS_PER_CU_DEFAULT)


def test_everything_dropped_and_outputs_given():
    M, K, N = 512, 512, 256
    X, W, dY = make_custom(M, K, N, "bf16", seed=9)
    print("bwd fused p=1", flush=True)
    m = sdrop.sdrop_mask(M, K, 128, 128, 1.0, 0, 0)
    dx = torch.full((M, K), 7.0, dtype=torch.bfloat16, device="cuda")
    dw = torch.full((K, N), 7.0, dtype=torch.bfloat16, device="cuda")
    a, b = sdrop.sdrop_bwd(dY.cuda(), W.cuda(), X.cuda(), m, out_dx=dx, out_dw=dw)
    torch.cuda.synchronize()
    assert a is dx and b is dw
    for o in (dx, dw):
        assert torch.count_nonzero(o).item() == 0 and not torch.signbit(o).any().item()


@pytest.mark.parametrize("width", [128, 256])
def test_one_launch_for_64_blocks_with_either_dx_tile_width(width):
    M, K, N, B, p, seed = 1024, 768, 512, 64, 0.4, 21
    print("bwd fused 64-blocks width", width, flush=True)
    X, W, dY = make_custom(M, K, N, "bf16", seed=seed)
    m = sdrop.sdrop_mask(M, K, B, B, p, seed, 0)
    keep = orc.mask(M // B, K // B, p, seed, 0)
    Xg, Wg, dYg = X.cuda(), W.cuda(), dY.cuda()
    sdrop.set_tuning(sdrop.TUNE_DX_TILE_WIDTH, width)
    try:
        dx, dw = sdrop.sdrop_bwd(dYg, Wg, Xg, m, out_dtype=torch.float32)
        assert torch.equal(dx, sdrop.sdrop_bwd_dx(dYg, Wg, m, out_dtype=torch.float32))
        assert torch.equal(dw, sdrop.sdrop_bwd_dw(Xg, dYg, m, out_dtype=torch.float32))
    finally:
        sdrop.set_tuning(sdrop.TUNE_DX_TILE_WIDTH, 0)
    assert_close(f64(dx), orc.bwd_dx(f64(dY), f64(W), keep, B, B, p), "dX 64-blocks width %d" % width)
    assert_close(f64(dw), orc.bwd_dw(f64(X), f64(dY), keep, B, B, p), "dW 64-blocks width %d" % width)


@pytest.mark.parametrize("M,K,N,p,dtype,ld", [
    (1536, 1536, 512, 0.0, "bf16", 0),      # dX on single blocks: no copy, both in place; dW's parts summed in the accumulators
    (2560, 2560, 1024, 0.0, "bf16", 0),     # the copy; dW's parts summed in the accumulators
    (2560, 2560, 256, 0.1, "f16", 0),       # dW in parts, planes and a summing pass
    (2560, 2688, 256, 0.1, "bf16", 24),     # an odd number of block columns, row-strided operands
    (4096, 2560, 2816, 0.2, "bf16", 0),     # both in place, dW in one part
    (4096, 4096, 2048, 0.1, "bf16", 0),     # the copy; as many dW tiles as CUs: one part
])
def test_nk_weight_through_a_copy_in_one_launch(M, K, N, p, dtype, ld):
    """dX on tiles of two blocks reads a transposed copy of W[N,K] while dW is written as [N,K] in the same launch."""
    print("bwd fused nk copy", M, K, N, p, dtype, ld, flush=True)
    X, W, dY = make_custom(M, K, N, dtype, seed=23)
    m = sdrop.sdrop_mask(M, K, 128, 128, p, 9, 0)

    def strided(t):
        t = t.cuda()
        if ld == 0:
            return t.contiguous()
        wide = torch.zeros(t.shape[0], t.shape[1] + ld, dtype=t.dtype, device="cuda")
        wide[:, :t.shape[1]] = t
        return wide[:, :t.shape[1]]

    Xg, Wnk, dYg = strided(X), strided(W.t()), strided(dY)
    for out_dtype in (torch.float32, None):
        ref_dx = sdrop.sdrop_bwd_dx(dY.cuda(), W.cuda(), m, out_dtype=out_dtype)
        ref_dw = sdrop.sdrop_bwd_dw(X.cuda(), dY.cuda(), m, out_dtype=out_dtype)
        try:
            for fused in (1, 0):
                sdrop.set_tuning(sdrop.TUNE_BWD_FUSED, fused)
                dx, dw = sdrop.sdrop_bwd(dYg, Wnk, Xg, m, out_dtype=out_dtype, w_layout=sdrop.W_NK)
                torch.cuda.synchronize()
                assert torch.equal(dx, ref_dx) and torch.equal(dw, ref_dw.t()), (fused, out_dtype)
        finally:
            sdrop.set_tuning(sdrop.TUNE_BWD_FUSED, 1)


class _KernelNode(ctypes.Structure):        # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _launches(f):
    """Workgroups of each launch that a call records into a graph, in the order of the graph's nodes (nothing runs)."""
    f()                                                 # (modules loaded, attributes set)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    s = torch.cuda.Stream()
    with torch.cuda.graph(g, stream=s):
        f()
    L, n, node = sdrop.lib(), ctypes.c_size_t(0), _KernelNode()      # (the HIP runtime that the library is linked to)
    L.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    L.hipGraphKernelNodeGetParams.argtypes = [ctypes.c_void_p, ctypes.POINTER(_KernelNode)]
    assert L.hipGraphGetNodes(g.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert L.hipGraphGetNodes(g.raw_cuda_graph(), nodes, ctypes.byref(n)) == 0
    grids = []
    for i in range(n.value):
        assert L.hipGraphKernelNodeGetParams(nodes[i], ctypes.byref(node)) == 0
        grids.append(node.grid[0] * node.grid[1] * node.grid[2])
    return grids


@pytest.mark.parametrize("M,K,N,p,groups,launches", [
    (4736, 14336, 256, 0.0, None, 1),       # dX tiles of two blocks on the persistent kernel, dW's parts summed in the accumulators
    (2560, 2560, 1024, 0.1, 0, 1),          # the same form forced at a smaller size
    (2560, 2560, 1024, 0.1, None, 1),       # dX a workgroup per tile of two blocks, the same dW
    (1536, 1536, 512, 0.0, None, 1),        # dX on single blocks
    (2560, 2560, 256, 0.1, 0, 2),           # dW in parts: the summing pass follows
])
def test_one_call_is_one_launch(M, K, N, p, groups, launches):
    print("bwd launches", M, K, N, p, groups, flush=True)
    X, W, dY = (torch.randn(s, device="cuda").to(torch.bfloat16) for s in ((M, K), (K, N), (M, N)))
    m = sdrop.sdrop_mask(M, K, 128, 128, p, 3, 0)
    dx, dw = torch.empty_like(X), torch.empty_like(W)
    ws = torch.empty(max(sdrop.workspace_bytes(sdrop.OP_BWD_DW, M, K, N, 128, 128, X.dtype, X.dtype), 16), dtype=torch.uint8, device="cuda")
    if groups is not None:
        sdrop.set_tuning(sdrop.TUNE_DX_PERSISTENT_GROUPS_PER_CU, groups)
    try:
        assert len(_launches(lambda: sdrop.sdrop_bwd(dY, W, X, m, out_dx=dx, out_dw=dw, ws=ws))) == launches
        assert torch.equal(dx, sdrop.sdrop_bwd_dx(dY, W, m)) and torch.equal(dw, sdrop.sdrop_bwd_dw(X, dY, m, ws=ws))
    finally:
        sdrop.set_tuning(sdrop.TUNE_DX_PERSISTENT_GROUPS_PER_CU, sdrop.DX_PERSISTENT_GROUPS_PER_CU_DEFAULT)


@pytest.mark.parametrize("M,K,N,dw_groups", [
    (256, 512, 512, 8),         # dX's reduction is the longer one: dW on 128 x 256 tiles
    (512, 512, 512, 16),        # no longer than dW's: 128 x 128 tiles
    (512, 512, 768, 12),
    (768, 512, 768, 24),
])
def test_tiles_of_a_list_of_one_part(M, K, N, dw_groups):
    print("bwd one part", M, K, N, flush=True)
    X, W, dY = (torch.randn(s, device="cuda").to(torch.bfloat16) for s in ((M, K), (K, N), (M, N)))
    m = sdrop.sdrop_mask(M, K, 128, 128, 0.0, 3, 0)
    dx, dw = torch.empty_like(X), torch.empty_like(W)
    grids = _launches(lambda: sdrop.sdrop_bwd(dY, W, X, m, out_dx=dx, out_dw=dw))
    assert grids == [(M // 128) * (K // 128) + dw_groups]       # a workgroup for each of dX's blocks, and dW's
    assert torch.equal(dx, sdrop.sdrop_bwd_dx(dY, W, m)) and torch.equal(dw, sdrop.sdrop_bwd_dw(X, dY, m))


@pytest.mark.parametrize("M,K,N,p,launches", [
    (8192, 1024, 512, 0.2, 3),          # the weight's copy, both gradients, the sum of dW's parts
    (16384, 512, 512, 0.0, 4),          # the copy, dX, dW's parts on narrow tiles, their sum
    (16384, 1024, 512, 0.2, 3),         # as long, but dW alone would take wide tiles
    (10240, 512, 256, 0.0, 3),          # as long and narrow, but all of it fits the chip at once
])
def test_launches_with_an_nk_weight_through_a_copy(M, K, N, p, launches):
    print("bwd launches nk", M, K, N, p, flush=True)
    X, W, dY = (torch.randn(s, device="cuda").to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    m = sdrop.sdrop_mask(M, K, 128, 128, p, 3, 0)
    dx, dw = torch.empty_like(X), torch.empty_like(W)
    need = sdrop.workspace_bytes(sdrop.OP_BWD_DW, M, K, N, 128, 128, X.dtype, X.dtype, sdrop.W_NK)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert len(_launches(lambda: sdrop.sdrop_bwd(dY, W, X, m, out_dx=dx, out_dw=dw, ws=ws, w_layout=sdrop.W_NK))) == launches
    Wk = W.t().contiguous()
    assert torch.equal(dx, sdrop.sdrop_bwd_dx(dY, Wk, m)) and torch.equal(dw.t(), sdrop.sdrop_bwd_dw(X, dY, m))
