"""SparseDropLinear's place in an autograd graph: what a step keeps, and which gradients of the bias go through the library.

The library's calls are stood in for by dense products on the CPU (with nothing dropped), so only the wiring of autograd.py
is under test: eq. (1)-(3) of arxiv 2411.01238, Section 3.1, with the layer's own bias behind them."""
import pytest
import torch
from torch.autograd import forward_ad

from paper_2411_01238_amd import autograd, sdrop


class _Layer(autograd.SparseDropLinear):
    def __init__(self, K, N, dtype=torch.float32):
        super().__init__(K, N, p=0.0, BM=64, BK=64, bias=True, dtype=dtype, device="cpu")


@pytest.fixture
def summed(monkeypatch):
    """Dense stand-ins; returns the list of the tensors that the column-sum kernel was given."""
    seen = []

    def fwd(x, w, BM, BK, p, seed, rng_stream=0, w_layout=sdrop.W_KN, bias=None, **kw):
        y = x.detach() @ w.detach()
        return (y if bias is None else y + bias.detach()), "a mask"

    def col_sum(dy):
        assert dy.data_ptr() % 16 == 0              # (what the kernel's 16-byte loads need; raises where there is no memory)
        seen.append(dy)
        return dy.detach().sum(0)

    monkeypatch.setattr(sdrop, "sdrop_fwd_seeded", fwd)
    monkeypatch.setattr(sdrop, "sdrop_bwd", lambda dy, w, x, m, w_layout: (dy @ w.t(), x.t() @ dy))
    monkeypatch.setattr(sdrop, "sdrop_bwd_dx_ex", lambda dy, w, m, w_layout: dy @ w.t())
    monkeypatch.setattr(sdrop, "sdrop_bwd_dw_ex", lambda x, dy, m, w_layout: x.t() @ dy)
    monkeypatch.setattr(sdrop, "sdrop_col_sum", col_sum)
    return seen


def test_a_step_that_trains_the_bias_alone_keeps_no_operand(summed):
    layer = _Layer(64, 8)
    layer.weight.requires_grad_(False)
    kept = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: kept.append(t) or t, lambda t: t):
        y = layer(torch.randn(64, 64))
    assert not kept and getattr(y.grad_fn, "mask", None) is None
    dy = torch.randn(64, 8)
    (db,) = torch.autograd.grad(y, [layer.bias], dy)
    assert torch.equal(db, dy.sum(0)) and len(summed) == 1


def test_gradients_of_a_whole_step(summed):
    layer, x, dy = _Layer(64, 8), torch.randn(64, 64, requires_grad=True), torch.randn(64, 8)
    dx, dw, db = torch.autograd.grad(layer(x), [x, layer.weight, layer.bias], dy)
    assert torch.equal(dx, dy @ layer.weight.t()) and torch.equal(dw, x.t() @ dy) and torch.equal(db, dy.sum(0))
    assert len(summed) == 1


def test_gradients_the_kernel_cannot_read_are_summed_by_torch(summed):
    layer = _Layer(64, 8)
    x = torch.randn(64, 64)
    # a gradient whose memory is not 16-byte aligned
    wide = torch.randn(64 * 8 + 1)
    dy = wide[1:].view(64, 8)
    assert dy.data_ptr() % 16 != 0
    assert torch.equal(torch.autograd.grad(layer(x), [layer.bias], dy)[0], dy.sum(0))
    # several gradients at once
    dys = torch.randn(3, 64, 8)
    (db,) = torch.autograd.grad(layer(x), [layer.bias], dys, is_grads_batched=True)
    assert torch.allclose(db, dys.sum(1))
    # a gradient that carries a tangent
    y = layer(x)
    with forward_ad.dual_level():
        (db,) = torch.autograd.grad(y, [layer.bias], forward_ad.make_dual(dys[0], dys[1]))
        tangent = forward_ad.unpack_dual(db).tangent
        assert tangent is not None and torch.allclose(tangent, dys[1].sum(0))
    # a gradient that is itself differentiated
    dy = dys[2].clone().requires_grad_(True)
    (db,) = torch.autograd.grad(layer(x), [layer.bias], dy, create_graph=True)
    assert torch.equal(torch.autograd.grad(db.sum(), [dy])[0], torch.ones_like(dy))
    assert not summed
