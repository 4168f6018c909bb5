"""What a user of this library has it do, as a list of timed cases.

A case is one pass of one of the library's public paths:

    step     one training step of a layer through the binding, as bench.py runs it: the mask and eq. (1) by
             sdrop_fwd_seeded, eq. (2) and (3) by sdrop_bwd, into outputs, a mask object and a workspace that the
             program keeps
    linear   SparseDropLinear in a training loop: forward, and backward through autograd
    block    sparse_act_block (Linear -> activation -> SparseDrop -> Linear, every product sparse): forward and
             backward through autograd
    eval     SparseDropLinear in eval mode, forward only (nothing is dropped)

M x K is the activation in front of the dropped layer (rows x features), N the layer's outputs, BM x BK the mask
block; a block case has N0 features in front of its first layer.  Sizes are those of workloads.py, of the models in
model_step.py (width 1024; 1024-row MLP batches, 4096-token GPT and 16384-token ViT batches) and of the tests.
"""
import math

import torch

from paper_2411_01238_amd import sdrop
from paper_2411_01238_amd.autograd import SparseDropLinear, sparse_act_block

_DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, path, M, K, N, BM, BK, p, dtype, out="", layout="kn", bias=False, act="", N0=0):
    c = {"path": path, "M": M, "K": K, "N": N, "BM": BM, "BK": BK, "p": p, "dtype": dtype}
    if name:
        c["name"] = name
    if path == "step":
        c["out"] = out or dtype
    if path in ("linear", "eval"):
        c["layout"], c["bias"] = layout, bias
    if path == "block":
        c["act"], c["N0"] = act, N0
    return c


def listed():
    return [
        # the smallest call of the tests and the smoke run: launches and the host path are all of it
        _case("tiny_step", "step", 256, 256, 256, 64, 64, 0.5, "f16"),
        # a hidden layer of the MLP at its own batch size, as its training loop calls it
        _case("mlp_linear_1024", "linear", 1024, 1024, 1024, 128, 128, 0.5, "bf16"),
        # one layer of the stacked MLP-classifier workload: small blocks, a short reduction
        _case("mlp_step", "step", 8192, 1024, 1024, 64, 64, 0.5, "f16"),
        # gradients kept in fp32 (accumulation over micro-batches), medium size
        _case("f32_grads_step", "step", 2048, 2048, 2048, 128, 128, 0.3, "bf16", out="f32"),
        # the benchmark's headline and the light-dropout end of its sweep
        _case("square_half_step", "step", 4096, 4096, 4096, 128, 128, 0.5, "bf16"),
        _case("square_tenth_step", "step", 4096, 4096, 4096, 128, 128, 0.1, "bf16"),
        # the output layer of the character GPT: 72 columns, a ragged edge in every product
        _case("gpt_head_linear", "linear", 4096, 1024, 72, 128, 128, 0.3, "bf16"),
        # the query-key-value projection of the ViT with torch.nn.Linear's weight layout and a bias
        _case("vit_qkv_linear_nk", "linear", 16384, 1024, 3072, 128, 128, 0.2, "bf16", layout="nk", bias=True),
        # the feed-forward block of the GPT with both layers sparse
        _case("gpt_ffn_gelu_block", "block", 4096, 4096, 1024, 128, 128, 0.5, "bf16", act="gelu", N0=1024),
        # the transformer down-projection workload: blocks of unequal sides, light dropout
        _case("ffn_down_step", "step", 16384, 3072, 768, 128, 64, 0.1, "bf16"),
        # inference of a 1000-way classifier layer: forward only, N not a multiple of the tile
        _case("classifier_eval", "eval", 8192, 1024, 1000, 64, 64, 0.5, "f16", bias=True),
        # the large skinny workload
        _case("skinny_step", "step", 65536, 4096, 1024, 128, 128, 0.3, "bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _cost(c):
    gemms = {"step": 3, "linear": 3, "block": 6, "eval": 1}[c["path"]]
    return gemms * c["M"] * c["K"] * max(c["N"], c.get("N0", 0))


def draw(rng):
    """One more case: the paths, data types, blocks and rates of the listed ones over the range of sizes between them."""
    largest = max(_cost(c) for c in listed())
    while True:
        path = rng.choice(("step", "step", "step", "linear", "linear", "block", "eval"))
        BM, BK = rng.choice(((128, 128), (128, 128), (64, 64), (128, 64)))
        M = max(1, round(_log_uniform(rng, 256, 65536) / BM)) * BM
        K = max(1, round(_log_uniform(rng, 256, 4096) / BK)) * BK
        N = _log_uniform(rng, 64, 4096)
        # layer widths are mostly whole multiples of a tile; class counts and vocabularies are not
        N = max(1, round(N / 256)) * 256 if rng.random() < 0.5 else max(8, round(N / 8)) * 8
        p = rng.choice((0.1, 0.2, 0.3, 0.5, 0.7))
        dtype = rng.choice(("bf16", "bf16", "f16"))
        c = _case("", path, M, K, N, BM, BK, p, dtype, out=rng.choice((dtype, dtype, "f32")),
                  layout=rng.choice(("kn", "nk")), bias=rng.random() < 0.5, act=rng.choice(("relu", "gelu", "gelu_tanh")), N0=N)
        if _cost(c) <= largest:
            return c


def _normal(shape, g, std, dtype):
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=g).to(dtype)


def prepare(case, seed):
    M, K, N, BM, BK, p = (case[k] for k in ("M", "K", "N", "BM", "BK", "p"))
    dt = _DT[case["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    s = {"case": case, "seed": seed}
    if case["path"] == "step":
        out = _DT[case["out"]]
        s["X"], s["W"], s["dY"] = _normal((M, K), g, 1.0, dt), _normal((K, N), g, K ** -0.5, dt), _normal((M, N), g, 1.0, dt)
        s["Y"], s["dX"], s["dW"] = (torch.empty(shape, dtype=out, device="cuda") for shape in ((M, N), (M, K), (K, N)))
        s["mask"] = sdrop.Mask(M, K, BM, BK, p)
        need = sdrop.workspace_bytes(sdrop.OP_BWD_DW, M, K, N, BM, BK, dt, out)
        s["ws"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    elif case["path"] in ("linear", "eval"):
        train = case["path"] == "linear"
        s["layer"] = SparseDropLinear(K, N, p, BM, BK, bias=case["bias"], seed=seed, dtype=dt, weight_layout=case["layout"])
        with torch.no_grad():
            s["layer"].weight.copy_(_normal(s["layer"].weight.shape, g, K ** -0.5, dt))
            if case["bias"]:
                s["layer"].bias.copy_(_normal((N,), g, 0.1, dt))
        s["layer"].train(train)
        s["X"] = _normal((M, K), g, 1.0, dt).requires_grad_(train)
        if train:
            s["dY"] = _normal((M, N), g, 1.0, dt)
    else:
        N0 = case["N0"]
        s["H"], s["W0"], s["b0"] = _normal((M, N0), g, 1.0, dt), _normal((K, N0), g, N0 ** -0.5, dt), _normal((K,), g, 0.1, torch.float32)
        s["W"], s["dY"] = _normal((K, N), g, K ** -0.5, dt), _normal((M, N), g, 1.0, dt)
        for k in ("H", "W0", "b0", "W"):
            s[k].requires_grad_(True)
    return s


def run(s):
    c = s["case"]
    if c["path"] == "step":
        sdrop.sdrop_fwd_seeded(s["X"], s["W"], c["BM"], c["BK"], c["p"], s["seed"], 0, mask=s["mask"], out_dtype=s["Y"].dtype, out=s["Y"])
        sdrop.sdrop_bwd(s["dY"], s["W"], s["X"], s["mask"], out_dtype=s["dX"].dtype, out_dx=s["dX"], out_dw=s["dW"], ws=s["ws"])
        return {"Y": s["Y"], "dX": s["dX"], "dW": s["dW"]}
    if c["path"] == "eval":
        with torch.no_grad():
            return s["layer"](s["X"])
    if c["path"] == "linear":
        y = s["layer"](s["X"])
        wanted = [s["X"]] + list(s["layer"].parameters())
    else:
        y = sparse_act_block(s["H"], s["W0"], s["b0"], s["W"], c["p"], c["act"], c["BM"], c["BK"], s["seed"], 0)
        wanted = [s[k] for k in ("H", "W0", "b0", "W")]
    return [y.detach()] + list(torch.autograd.grad(y, wanted, s["dY"]))


def work(case):
    """Each input read once (of X the kept blocks only), each output written once; the products over kept blocks."""
    M, K, N, f = case["M"], case["K"], case["N"], 1.0 - case["p"]
    out = 4 if case.get("out") == "f32" else 2
    if case["path"] == "eval":
        return {"bytes": 2.0 * (M * K + K * N + M * N), "flops": 2.0 * M * K * N}
    if case["path"] == "block":
        N0 = case["N0"]
        read = 2 * (M * N0 + K * N0 + K * N + M * N) + 4 * K
        written = 2 * (M * N + M * N0 + K * N0 + K * N) + 4 * K
        return {"bytes": float(read + written), "flops": 6.0 * f * M * K * (N0 + N)}
    return {"bytes": 2.0 * (f * M * K + K * N + M * N) + out * (M * N + M * K + K * N), "flops": 6.0 * f * M * K * N}


def tolerance(case):
    """About four times the 2-norm error of each path against the same products in float64 on the same 16-bit inputs:
    1.7e-3 (bf16) and 2.1e-4 (fp16) where the result is rounded once, 2.4e-3 and 3.0e-4 with a bias (two roundings) or
    in a block (hidden values are rounded as well), 6.4e-4 in an fp16 block with a ReLU (a hidden value near 0 may fall on
    either side of the gate); fp32 results, sums over 2048 products, 2.7e-7, and the error grows with the square root of
    the length (65536: 1.0e-6)."""
    if case.get("out") == "f32":
        return {"rel": 4e-6}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": 2.5e-3} if case["path"] == "block" else {"rel": 1.2e-3}
