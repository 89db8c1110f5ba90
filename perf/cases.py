"""Performance cases of the fallback-quantization library: the work a training or evaluation program
has it do, through the public Python entry points, over the range of shapes it is used on.

Kinds of pass
  forward   quantize the activation X (bf16, run-time fallback) and multiply with the weight that the
            program keeps quantized: Y = X W^T
  backward  the gradient recipe: dY with stochastic rounding (or with fallback), dX = dY W and
            dW = dY^T X on the transposed code copies
  step      one training step of a linear layer: the weight, which the optimizer has just changed, X and
            its stored context, the forward product, dY and the two backward products
  glu       SiLU-gated linear unit, forward with both INT10 contexts and backward from them
  rmsnorm   RMS normalization, forward with its INT10 context and backward from it

A case's sizes: M tokens (rows), K input features, N output features (glu and rmsnorm: M rows, K columns).
`fb` is the fraction of X's (or dY's) 128 x 128 blocks that hold outliers and fall back.
"""
import math

import torch

import paper_2503_08040_amd as fq

BLOCK = 128
OUT = {"bf16": torch.bfloat16, "f32": torch.float32}

# The largest listed product, in multiply-adds: a drawn case stays below it.
MAX_MACS = 8192 ** 3
MAX_ELEMENTS = 4096 * 11008


def listed():
    return [
        # the smallest layer the benchmark names: launches and latency are all there is
        {"name": "forward_small", "kind": "forward", "M": 256, "K": 512, "N": 512, "fb": 0.125,
         "data": "normal", "out": "f32", "variant": "exact"},
        # its backward, with fallback on a heavy-tailed gradient
        {"name": "backward_small", "kind": "backward", "M": 256, "K": 512, "N": 512, "fb": 0.25,
         "out": "f32", "rounding": "nearest"},
        # evaluation of a handful of tokens: the weight's bytes are the work
        {"name": "forward_few_tokens", "kind": "forward", "M": 33, "K": 4096, "N": 11008, "fb": 0.05,
         "data": "normal", "out": "bf16", "variant": "exact"},
        # a ragged batch through a layer whose sizes are no multiples of the block
        {"name": "forward_ragged", "kind": "forward", "M": 777, "K": 1544, "N": 2200, "fb": 0.05,
         "data": "normal", "out": "bf16", "variant": "exact"},
        # GLU up / gate projection of a full batch, the benchmark's default workload
        {"name": "forward_up", "kind": "forward", "M": 4096, "K": 4096, "N": 11008, "fb": 0.05,
         "data": "normal", "out": "bf16", "variant": "exact"},
        # GLU down projection: outliers along whole channels of silu(a) * b
        {"name": "forward_down", "kind": "forward", "M": 4096, "K": 11008, "N": 4096, "fb": 0.047,
         "data": "glu", "out": "bf16", "variant": "exact"},
        # the same kind of layer in a smaller batch through the tolerance variant of the product
        {"name": "forward_biased", "kind": "forward", "M": 2048, "K": 4096, "N": 4096, "fb": 0.05,
         "data": "normal", "out": "bf16", "variant": "biased"},
        # the square problem in the middle of the fallback range that training runs at
        {"name": "forward_square", "kind": "forward", "M": 8192, "K": 8192, "N": 8192, "fb": 0.2,
         "data": "normal", "out": "bf16", "variant": "exact"},
        # backward of the up projection
        {"name": "backward_up", "kind": "backward", "M": 4096, "K": 4096, "N": 11008, "fb": 0.0,
         "out": "bf16", "rounding": "stochastic"},
        # a whole training step of a small layer
        {"name": "step_2048", "kind": "step", "M": 2048, "K": 2048, "N": 2048, "fb": 0.2,
         "out": "bf16"},
        # the non-linear layers around the projections
        {"name": "glu", "kind": "glu", "M": 4096, "K": 11008},
        {"name": "rmsnorm", "kind": "rmsnorm", "M": 4096, "K": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tokens(rng, lo, hi):
    """A number of tokens: any number, or a multiple of the block."""
    m = _log_int(rng, lo, hi)
    return m if rng.random() < 0.6 else max(BLOCK, m // BLOCK * BLOCK)


def _features(rng, lo, hi):
    """A feature dimension: mostly a multiple of the block, sometimes of 8 only, rarely odd."""
    n, kind = _log_int(rng, lo, hi), rng.random()
    if kind < 0.6:
        return max(BLOCK, n // BLOCK * BLOCK)
    return max(8, n // 8 * 8) if kind < 0.9 else n | 1


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "backward", "step", "glu", "rmsnorm"])
    if kind in ("glu", "rmsnorm"):
        while True:
            case = {"kind": kind, "M": _tokens(rng, 16, 8192), "K": _features(rng, 256, 11008)}
            if case["M"] * case["K"] <= MAX_ELEMENTS:
                return case
    products = {"forward": 1, "backward": 2, "step": 3}[kind]
    while True:
        M = _tokens(rng, 16 if kind == "forward" else 128, 8192)
        K, N = _features(rng, 256, 11008), _features(rng, 256, 11008)
        if products * M * K * N <= 0.8 * MAX_MACS:
            break
    case = {"kind": kind, "M": M, "K": K, "N": N, "fb": round(rng.uniform(0.0, 0.3), 3),
            "out": rng.choice(["bf16", "bf16", "f32"])}
    if kind == "forward":
        case["data"] = rng.choice(["normal", "glu"])
        case["variant"] = rng.choice(["exact", "exact", "exact", "biased"])
    elif kind == "backward":
        case["rounding"] = rng.choice(["stochastic", "stochastic", "nearest"])
        if case["rounding"] == "stochastic":
            case["fb"] = 0.0
    return case


# ---- inputs ---------------------------------------------------------------------------------------


def _randn(g, *shape):
    return torch.randn(shape, device="cuda", generator=g, dtype=torch.float32)


def _rand(g, *shape):
    return torch.rand(shape, device="cuda", generator=g, dtype=torch.float32)


def _blocks(n):
    return -(-n // BLOCK)


def _activation(g, M, K, fb, data):
    """(X bf16, theta).  "normal": N(0, 1), the outlier blocks hold one to four sparse channels of
    magnitude 50 to 200.  "glu": silu(a) * b with channels x100 along all tokens."""
    nbr, nbc = _blocks(M), _blocks(K)
    if data == "glu":
        a = _randn(g, M, K)
        x = torch.nn.functional.silu(a).mul_(_randn(g, M, K))
        n = int(round(fb * nbc)) if fb * nbc >= 0.5 or fb == 0 else 1
        cols = torch.randperm(nbc, device="cuda", generator=g)[:n] * BLOCK
        cols = (cols + (_rand(g, n) * BLOCK).long()).clamp_(max=K - 1)
        x[:, cols] *= 100.0
        return x.to(torch.bfloat16), 30.0
    x = _randn(g, M, K)
    n = int(round(fb * nbr * nbc))
    if n:
        ids = torch.randperm(nbr * nbc, device="cuda", generator=g)[:n]
        bi, bk = ids // nbc, ids % nbc
        width = (K - bk * BLOCK).clamp(max=BLOCK)
        # four distinct channels inside the block, one to four of them in use
        order = _rand(g, n, BLOCK) + 2.0 * (torch.arange(BLOCK, device="cuda")[None, :] >= width[:, None])
        chan = order.argsort(dim=1)[:, :4]
        used = torch.arange(4, device="cuda")[None, :] < 1 + (_rand(g, n, 1) * 4).long()
        used = used & (chan < width[:, None])
        hit = _rand(g, n, 4, BLOCK) < 0.25
        hit[:, 0, 0] = True
        rows = (bi * BLOCK)[:, None, None] + torch.arange(BLOCK, device="cuda")[None, None, :]
        keep = hit & used[:, :, None] & (rows < M)
        cols = (bk[:, None] * BLOCK + chan)[:, :, None].expand(n, 4, BLOCK)
        value = (50.0 + 150.0 * _rand(g, n, 4, BLOCK)) * torch.where(_rand(g, n, 4, BLOCK) < 0.5, -1.0, 1.0)
        rows = rows.expand(n, 4, BLOCK)
        x[rows[keep], cols[keep]] = value[keep]
    return x.to(torch.bfloat16), 10.0


def _weight(g, N, K):
    return (0.02 * _randn(g, N, K)).to(torch.bfloat16)


def _gradient(g, M, N):
    """Heavy-tailed: 1e-3 times Student's t with three degrees of freedom."""
    chi = _randn(g, M, N).square_()
    for _ in range(2):
        chi += _randn(g, M, N).square_()
    return (1e-3 * _randn(g, M, N) / (chi / 3.0).sqrt_()).to(torch.bfloat16)


def _threshold(x, fb):
    """The threshold under which the fraction fb of the blocks of x falls back, as the delayed
    threshold of earlier steps would have settled on."""
    M, N = x.shape
    pad = torch.nn.functional.pad(x.float().abs(), (0, -N % BLOCK, 0, -M % BLOCK))
    top = pad.view(_blocks(M), BLOCK, _blocks(N), BLOCK).amax(dim=(1, 3)).flatten().sort(descending=True).values
    n = min(int(round(fb * top.numel())), top.numel() - 1)
    return float(0.5 * (top[n - 1] + top[n])) if n > 0 else float(2 * top[0])


def _tensor(rows, cols, **kw):
    """A quantized tensor as a program keeps it from step to step (cleared: a list of flagged blocks
    is shorter than the space it has)."""
    q = fq.QTensor(rows, cols, **kw)
    q.storage.zero_()
    return q


def _seen(q):
    """What the quantizer writes for its caller."""
    fields = ["codes", "scales", "mask"] + (["fb_list"] if q.capacity else [])
    fields += ["codes_t"] if q.want_transposed else []
    return {f: q.view(f) for f in fields}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    kind, M, K = case["kind"], case["M"], case["K"]
    st = {"kind": kind}
    if kind == "glu":
        st["x1"], st["x2"], st["dy"] = (_randn(g, M, K).to(torch.bfloat16) for _ in range(3))
        return st
    if kind == "rmsnorm":
        st["x"], st["dy"] = (_randn(g, M, K).to(torch.bfloat16) for _ in range(2))
        st["w"] = (1.0 + 0.1 * _randn(g, K)).to(torch.bfloat16)
        return st
    N = case["N"]
    st["out"] = OUT[case["out"]]
    w = _weight(g, N, K)
    if kind == "forward":
        st["x"], st["theta"] = _activation(g, M, K, case["fb"], case["data"])
        st["qx"] = _tensor(M, K)
        st["qw"] = fq.fq_quantize(w, fq.FQ_CRIT_NONE, 0.0, capacity=0)
        st["product"] = fq.fq_gemm_biased if case["variant"] == "biased" else fq.fq_gemm
        st["seen"] = _seen(st["qx"])
        return st
    x, st["theta"] = _activation(g, M, K, case["fb"] if kind == "step" else 0.05, "normal")
    st["dy"], st["seed"] = _gradient(g, M, N), int(seed)
    if kind == "backward":
        st["qw"] = fq.fq_quantize(w, fq.FQ_CRIT_NONE, 0.0, capacity=0, want_transposed=True)
        st["qc"] = fq.fq_quantize_sr(x, int(seed) + 1, want_transposed=True)
        st["rounding"] = case["rounding"]
        if st["rounding"] == "nearest":
            st["theta"] = _threshold(st["dy"], case["fb"])
            st["qdy"] = _tensor(M, N, want_transposed=True)
        else:
            st["qdy"] = _tensor(M, N, capacity=0, want_transposed=True)
        st["seen"] = _seen(st["qdy"])
        return st
    st["x"], st["w"] = x, w
    st["qx"] = _tensor(M, K)
    st["qc"] = _tensor(M, K, capacity=0, want_transposed=True)
    st["qw"] = _tensor(N, K, capacity=0, want_transposed=True)
    st["qdy"] = _tensor(M, N, capacity=0, want_transposed=True)
    st["seen"] = {k: _seen(st[k]) for k in ("qx", "qc", "qw", "qdy")}
    return st


def run(st):
    kind = st["kind"]
    if kind == "forward":
        fq.fq_quantize(st["x"], fq.FQ_CRIT_ABSMAX_GT, st["theta"], out=st["qx"])
        y = st["product"](fq.FQ_OP_NT, st["qx"], st["qw"], out_dtype=st["out"])
        return y, st["seen"]
    if kind == "backward":
        if st["rounding"] == "stochastic":
            fq.fq_quantize_sr(st["dy"], st["seed"], out=st["qdy"])
        else:
            fq.fq_quantize(st["dy"], fq.FQ_CRIT_ABSMAX_GT, st["theta"], out=st["qdy"])
        dx = fq.fq_gemm(fq.FQ_OP_NN, st["qdy"], st["qw"], out_dtype=st["out"])
        dw = fq.fq_gemm(fq.FQ_OP_TN, st["qdy"], st["qc"], out_dtype=torch.float32)
        return dx, dw, st["seen"]
    if kind == "step":
        fq.fq_quantize(st["w"], fq.FQ_CRIT_NONE, 0.0, out=st["qw"])
        fq.fq_quantize(st["x"], fq.FQ_CRIT_ABSMAX_GT, st["theta"], out=st["qx"])
        y = fq.fq_gemm(fq.FQ_OP_NT, st["qx"], st["qw"], out_dtype=st["out"])
        fq.fq_quantize_sr(st["x"], st["seed"] + 1, out=st["qc"])
        fq.fq_quantize_sr(st["dy"], st["seed"], out=st["qdy"])
        dx = fq.fq_gemm(fq.FQ_OP_NN, st["qdy"], st["qw"], out_dtype=st["out"])
        dw = fq.fq_gemm(fq.FQ_OP_TN, st["qdy"], st["qc"], out_dtype=torch.float32)
        return y, dx, dw, st["seen"]
    if kind == "glu":
        y, ctx1, ctx2 = fq.fq_glu_forward(st["x1"], st["x2"])
        dx1, dx2 = fq.fq_glu_backward(st["dy"], ctx1, ctx2)
        return y, ctx1, ctx2, dx1, dx2
    y, rstd, ctx = fq.fq_rmsnorm_forward(st["x"], st["w"], 1e-6)
    dx, dw = fq.fq_rmsnorm_backward(st["dy"], ctx, rstd, st["w"])
    return y, rstd, ctx, dx, dw


def work(case):
    kind, M, K = case["kind"], case["M"], case["K"]
    e = M * K
    ctx = M * -(-K // 128) * 164            # one INT10 context: fields and scales
    if kind == "glu":                       # x1, x2 -> y, contexts; dy, contexts -> dx1, dx2
        return {"bytes": 6 * e + 2 * ctx + 2 * ctx + 6 * e, "flops": 20 * e}
    if kind == "rmsnorm":                   # x, w -> y, context; dy, context, w -> dx, dw
        return {"bytes": 4 * e + ctx + ctx + 4 * e + 8 * K + 8 * M, "flops": 12 * e}
    N, fb = case["N"], case["fb"]
    o = 2 if case["out"] == "bf16" else 4
    macs = M * N * K
    if kind == "forward":                   # X -> codes and residual codes; codes of W; Y
        return {"bytes": 2 * e + (1 + fb) * e + N * K + o * M * N, "flops": 2 * macs * (1 + fb)}
    grad = 2 * M * N + 2 * (1 + fb) * M * N   # dY -> codes in both orientations
    back = grad + N * K + o * e + e + 4 * N * K
    if kind == "backward":
        return {"bytes": back, "flops": 4 * macs * (1 + fb)}
    grad = 4 * M * N                        # no fallback on the gradient of a step
    back = grad + N * K + o * e + e + 4 * N * K
    fore = 2 * N * K + 2 * N * K + 2 * e + (1 + fb) * e + 2 * e + o * M * N
    return {"bytes": back + fore, "flops": 2 * macs * (3 + fb)}


def tolerance(case):
    """About four times what was measured: the biased product against the exact one (rel 1.6e-3, max
    8e-3), the non-linear layers against the same formulas in binary64 with the results rounded once
    (rel 4e-5, max one bf16 step)."""
    if case["kind"] in ("forward", "backward", "step"):
        if case.get("variant") == "biased":
            return {"rel": 6e-3, "max": 2.5e-2}
        # INT8 codes are whole numbers and the order of the products' binary32 terms is part of
        # the interface: another correct implementation gives the same bits
        return "exact"
    return {"rel": 1.6e-4, "max": 1.6e-2}
