"""torch.autograd wrapper over the binding: SparseDrop in front of a linear layer as one op.

Section 3.1 of arxiv 2411.01238: forward eq. (1), backward eq. (2) and (3), the block mask of
Section 3.2 drawn once per call and shared by the three products.  Everything runs in libsdrop's
kernels; this file only wires them into autograd (no arithmetic of its own besides the add of a bias that is not of
the operands' type, and the seed bookkeeping).
"""
import torch

from . import sdrop


def _kernel_readable(t):
    """May a kernel take a contiguous tensor's memory for its value?  A plain tensor with 16-byte aligned memory, outside
    forward-mode differentiation (a tangent would be lost); a batch of vmap has no memory of its own and says so."""
    if type(t) not in (torch.Tensor, torch.nn.Parameter) or torch.autograd.forward_ad._current_level >= 0:
        return False
    try:
        return t.data_ptr() % 16 == 0
    except RuntimeError:
        return False


class _SparseDropMatmul(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, w, bias, p, BM, BK, seed, rng_stream, w_layout, inference):
        if inference and p == 0.0 and sdrop.fwd_dense_has_kernel(x, w, w_layout):
            # nothing is dropped and no backward follows: the product without a mask, where there is a kernel for it (a call
            # that comes back with none takes 6 us of a small layer's 19, so the shape is looked at first)
            y = sdrop.sdrop_fwd_dense(x, w, BM, BK, w_layout=w_layout, bias=bias)
            if y is not None:
                return y
        # the mask and eq. (1), plus the bias if there is one, in one call (one launch for block grids up to 128 x 64);
        # m serves the backward
        y, m = sdrop.sdrop_fwd_seeded(x, w, BM, BK, p, seed, rng_stream, w_layout=w_layout, bias=bias)
        # (a step that trains the bias alone needs none of these)
        if ctx.needs_input_grad[0] or ctx.needs_input_grad[1]:
            ctx.save_for_backward(x, w)
            ctx.mask = m
        ctx.w_layout = w_layout
        return y

    @staticmethod
    def backward(ctx, dy):
        if ctx.needs_input_grad[0] or ctx.needs_input_grad[1]:
            x, w = ctx.saved_tensors
        dy = dy.contiguous()
        wl = ctx.w_layout
        if ctx.needs_input_grad[0] and ctx.needs_input_grad[1]:
            dx, dw = sdrop.sdrop_bwd(dy, w, x, ctx.mask, w_layout=wl)      # both gradients, one launch where the shapes allow it
        else:
            dx = sdrop.sdrop_bwd_dx_ex(dy, w, ctx.mask, w_layout=wl) if ctx.needs_input_grad[0] else None
            dw = sdrop.sdrop_bwd_dw_ex(x, dy, ctx.mask, w_layout=wl) if ctx.needs_input_grad[1] else None
        db = None
        if ctx.needs_input_grad[2]:
            # (as a torch operation where the caller differentiates the gradient once more, it is linear in dy, and where dy
            # is not memory that the kernel can read)
            db = dy.sum(0) if (torch.is_grad_enabled() and dy.requires_grad) or not _kernel_readable(dy) else sdrop.sdrop_col_sum(dy)
        return dx, dw, db, None, None, None, None, None, None, None


def sparsedrop_matmul(x, w, p, BM=128, BK=128, seed=0, rng_stream=0, weight_layout="kn"):
    """y = (x . m') w / (1 - p) with a fresh block mask m' (Bernoulli(1-p) per BM x BK block of x).

    x [M, K] and w [K, N] are fp16 / bf16 GPU tensors with contiguous rows; M % BM == 0, K % BK == 0, N % 8 == 0.
    weight_layout="nk": w is [N, K], one row per output feature (the layout of torch.nn.Linear's weight), and so is
    its gradient.
    """
    wl = {"kn": sdrop.W_KN, "nk": sdrop.W_NK}[weight_layout]
    return _SparseDropMatmul.apply(x, w, None, float(p), int(BM), int(BK), int(seed), int(rng_stream), wl, not torch.is_grad_enabled())


def _fusable_bias(bias, x, n):
    """May the forward's kernel add this bias?  A plain vector of x's type, as the kernel reads it.  Anything else is added
    as a torch operation."""
    return (bias.dtype == x.dtype and bias.device == x.device and tuple(bias.shape) == (n,) and bias.is_contiguous()
            and _kernel_readable(bias))


_ACTS = {"relu": (sdrop.ACT_RELU, sdrop.GATE_RELU), "gelu_tanh": (sdrop.ACT_GELU_TANH, sdrop.GATE_GELU_TANH),
         "gelu": (sdrop.ACT_GELU_ERF, sdrop.GATE_GELU_ERF)}


class _SparseActBlock(torch.autograd.Function):
    """Linear -> activation -> SparseDrop -> Linear with every GEMM sparse (Section 4.3, closing remark).

    forward   X = m' . act(H W0^T + b0)          sdrop_producer (dropped blocks never computed;
                                                 for a GELU it also keeps Z = H W0^T + b0 on the kept blocks)
              Y = s X W                          eq. (1)
    backward  dZ  = s (dY W^T) . m' . act'(Z)    eq. (2) with the gate in its tail ([X > 0] for ReLU)
              dW  = s X^T dY                     eq. (3)
              dH  = dZ W0, dW0 = dZ^T H          eq. (1) / eq. (3) at scale 1 on the block-sparse dZ
              db0 = column sums of dZ            sdrop_bias_grad (kept blocks only)
    """

    @staticmethod
    def forward(ctx, h, w0, b0, w, p, BM, BK, seed, rng_stream, act):
        M, K = h.shape[0], w0.shape[0]
        act_id, gate_id = _ACTS[act]
        m = sdrop.sdrop_mask(M, K, BM, BK, p, seed, rng_stream)
        if act == "relu":
            x = sdrop.sdrop_producer(h, w0, b0, m, act=act_id)
            gate = x                    # [X > 0] is [Z > 0] on the kept blocks
        else:
            # (zero in the dropped blocks, which the gate does not read: the tensor is saved, and whoever looks at saved tensors
            # sees all of it)
            x, gate = sdrop.sdrop_producer(h, w0, b0, m, act=act_id, preact=True)
        y = sdrop.sdrop_fwd(x, w, m)
        ctx.save_for_backward(h, w0, w, x, gate)
        ctx.mask = m
        ctx.has_bias = b0 is not None
        ctx.gate_id = gate_id
        return y

    @staticmethod
    def backward(ctx, dy):
        h, w0, w, x, gate = ctx.saved_tensors
        m = ctx.mask
        dy = dy.contiguous()
        need_h, need_w0, need_b0, need_w = ctx.needs_input_grad[:4]
        dz = dh = dw0 = db0 = dw = None
        need_z = need_h or need_w0 or (need_b0 and ctx.has_bias)
        # products that do not depend on each other share a launch where both are wanted (contiguous matrices: row-strided
        # operands go through the calls that take leading dimensions)
        if need_z and need_w and all(t.is_contiguous() for t in (w, x, gate)):
            dz, dw = sdrop.sdrop_bwd_gated(dy, w, x, gate, ctx.gate_id, m)
        else:
            if need_z:
                dz = sdrop.sdrop_bwd_dx_ex(dy, w, m, relu_mask=gate, gate_mode=ctx.gate_id)
            if need_w:
                dw = sdrop.sdrop_bwd_dw(x, dy, m)
        if need_h and need_w0 and h.is_contiguous() and w0.is_contiguous():
            dh, dw0 = sdrop.sdrop_producer_bwd(dz, w0, h, m)
        else:
            if need_h:
                dh = sdrop.sdrop_fwd_ex(dz, w0, m, scale_mode=sdrop.SCALE_ONE)
            if need_w0:
                dw0 = sdrop.sdrop_bwd_dw_ex(dz, h, m, scale_mode=sdrop.SCALE_ONE)
        if need_b0 and ctx.has_bias:
            db0 = sdrop.sdrop_bias_grad(dz, m)
        return dh, dw0, db0, dw, None, None, None, None, None, None


def sparse_act_block(h, w0, b0, w, p, act="relu", BM=128, BK=128, seed=0, rng_stream=0):
    """y = s (m' . act(h w0^T + b0)) w with a fresh block mask m' over the hidden activation.

    h [M, N0], w0 [K, N0] (one row per hidden feature), b0 fp32 [K] or None, w [K, N]: contiguous
    fp16 / bf16 GPU tensors; M % BM == 0, K % BK == 0, N0 % 8 == 0, N % 8 == 0.
    act: "relu", "gelu" (the exact form) or "gelu_tanh".
    """
    return _SparseActBlock.apply(h, w0, b0, w, float(p), int(BM), int(BK), int(seed), int(rng_stream), act)


def sparse_relu_block(h, w0, b0, w, p, BM=128, BK=128, seed=0, rng_stream=0):
    """sparse_act_block with a ReLU."""
    return sparse_act_block(h, w0, b0, w, p, "relu", BM, BK, seed, rng_stream)


class SparseDropLinear(torch.nn.Module):
    """Dropout(p) followed by Linear(K -> N), with the dropout block-structured and fused into the
    layer's three GEMMs (the layer substitution of Section 4).  The weight is stored [K, N] as in
    Section 3.1, or, with weight_layout="nk", [N, K] like torch.nn.Linear's (a state dict of such a layer then loads
    as it is).  In eval mode nothing is dropped (p = 0: all blocks kept, scale 1)."""

    def __init__(self, in_features, out_features, p=0.5, BM=128, BK=128, bias=True, seed=0,
                 dtype=torch.bfloat16, device="cuda", weight_layout="kn"):
        super().__init__()
        self.p, self.BM, self.BK, self.seed = float(p), int(BM), int(BK), int(seed)
        if weight_layout not in ("kn", "nk"):
            raise ValueError("weight_layout is 'kn' or 'nk'")
        self.weight_layout = weight_layout
        w = torch.empty(in_features, out_features, dtype=torch.float32)
        torch.nn.init.kaiming_uniform_(w.t(), a=5 ** 0.5)
        if weight_layout == "nk":
            w = w.t().contiguous()
        self.weight = torch.nn.Parameter(w.to(dtype=dtype, device=device))
        self.bias = torch.nn.Parameter(torch.zeros(out_features, dtype=dtype, device=device)) if bias else None
        self.calls = 0          # the mask's rng_stream: a new mask every forward call

    def forward(self, x):
        # a matrix goes in as it is: a reshape of x and one of y would be two more nodes in the graph, which the backward
        # of a small layer feels (a 1024^3 layer is bound by its host time)
        matrix = x.dim() == 2
        x2 = (x if matrix else x.reshape(-1, x.shape[-1])).contiguous()
        p = self.p if self.training else 0.0
        nk = self.weight_layout == "nk"
        bias = self.bias
        if bias is not None and _fusable_bias(bias, x2, self.weight.shape[0 if nk else 1]):
            y = _SparseDropMatmul.apply(x2, self.weight, bias, p, self.BM, self.BK, self.seed, self.calls, sdrop.W_NK if nk else sdrop.W_KN,
                                         not torch.is_grad_enabled())
        else:
            y = sparsedrop_matmul(x2, self.weight, p, self.BM, self.BK, self.seed, self.calls, self.weight_layout)
            if bias is not None:
                y = y + bias
        if self.training:
            self.calls += 1
        return y if matrix else y.reshape(*x.shape[:-1], y.shape[-1])
