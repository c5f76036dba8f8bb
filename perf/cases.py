"""Cases on which the speed of the operators is measured, and how one pass of each is run.

A case names an operator, its sizes and the options of the entry point.  The listed ones stand for what a
decoder layer has this library do while it serves: blocks of a small model, decoding of a few tokens,
decoding of a batch, prefill of one and of many sequences, and the layer-norm projections and attention
beside them.  Inputs follow the recipes of bb_inputs.py (same distributions, drawn on the GPU).
"""
import math

import torch

import paper_2505_07829_amd as bb


def _ffn(name, M, D, F, x="normal", transposed=False, residual=False, eps=1e-5):
    return {"name": name, "op": "ffn", "M": M, "D": D, "F": F, "x": x, "transposed": transposed,
            "residual": residual, "eps": eps}


def _ln(name, M, D, N, transposed=False, eps=1e-5):
    return {"name": name, "op": "ln", "M": M, "D": D, "N": N, "transposed": transposed, "eps": eps}


def _attn(name, B, M, N, d, dv):
    return {"name": name, "op": "attention", "B": B, "M": M, "N": N, "d": d, "dv": dv}


def listed():
    return [
        # a small model's block on a short sequence: latency and launches
        _ffn("ffn_small", 64, 256, 704, eps=1e-6),
        # one decoding step for 16 sequences, heavy-tailed activations: the weight stream
        _ffn("ffn_decode", 16, 4096, 11008, x="student4", eps=1e-6),
        # one decoding step for 5 sequences of a checkpoint in linear-layer layout, with the block's residual
        _ffn("ffn_decode_linear_residual", 5, 4096, 11008, transposed=True, residual=True, eps=1e-6),
        # one decoding step for a hundred sequences: between the weight stream and the matrix cores
        _ffn("ffn_batch", 100, 4096, 11008),
        # prefill of one sequence
        _ffn("ffn_prefill", 2048, 4096, 11008),
        # prefill with a ragged number of tokens, model dimension no multiple of a tile, linear-layer layout, residual
        _ffn("ffn_prefill_linear_residual", 1000, 2880, 7680, transposed=True, residual=True),
        # prefill through a large block, activations with outlier channels
        _ffn("ffn_large", 4096, 8192, 28672, x="outlier_cols"),
        # the fused query/key/value projection behind a layer norm for a batch of decoding sequences
        _ln("ln_matmul_batch", 48, 4096, 12288),
        # the first product of a feed-forward block behind a layer norm, many tokens
        _ln("ln_matmul_large", 8192, 4096, 16384),
        # attention of a prefill: 32 heads, 4096 tokens
        _attn("attention_prefill", 32, 4096, 4096, 128, 128),
        # attention of one decoding step: one query per head
        _attn("attention_decode", 32, 1, 4096, 128, 128),
        # grouped-query decoding: 8 queries share the keys and values of each of 8 heads of 8 sequences, narrow heads
        _attn("attention_grouped", 64, 8, 5000, 64, 64),
    ]


# the work that bounds a drawn case: half of the largest listed one's operations, and its bytes
_MAX_FLOPS = 2.9e12
_MAX_BYTES = 1.4e9


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _rows(rng, hi):
    return max(1, min(hi, int(_log_uniform(rng, 1, hi + 1))))


def _dim(rng, lo, hi):
    """a model or hidden dimension: mostly a multiple of 64, now and then only of 8"""
    step = 64 if rng.random() < 0.8 else 8
    return max(step, int(_log_uniform(rng, lo, hi) / step + 0.5) * step)


def draw(rng):
    while True:
        kind = rng.choice(["ffn", "ffn", "ffn", "ln", "attention", "attention"])
        if kind == "ffn":
            D = _dim(rng, 256, 8192)
            case = _ffn("", _rows(rng, 4096), D, _dim(rng, 2 * D, 4 * D),
                        x=rng.choice(["normal", "student4", "outlier_cols"]), transposed=rng.random() < 0.4,
                        residual=rng.random() < 0.4, eps=rng.choice([1e-6, 1e-5]))
        elif kind == "ln":
            D = _dim(rng, 256, 8192)
            case = _ln("", _rows(rng, 8192), D, _dim(rng, D, 4 * D), transposed=rng.random() < 0.4)
        else:
            d = rng.choice([64, 128, 128])
            form = rng.choice(["prefill", "prefill", "decode", "grouped"])
            N = int(_log_uniform(rng, 64, 8192))
            # prefill: all tokens, or the last chunk of a longer sequence
            M = {"prefill": N if rng.random() < 0.5 else max(32, int(N * rng.uniform(0.1, 1.0))),
                 "decode": 1, "grouped": rng.choice([2, 4, 5, 8, 16])}[form]
            case = _attn("", max(4, int(_log_uniform(rng, 4, 128))), M, N, d, d)
        w = work(case)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES:
            del case["name"]
            return case


def _draw_x(gen, M, D, dist):
    x = torch.randn(M, D, generator=gen, device="cuda")
    if dist == "student4":
        chi2 = torch.zeros_like(x)
        for _ in range(4):
            chi2 += torch.randn(M, D, generator=gen, device="cuda") ** 2
        x /= torch.sqrt(chi2 / 4.0)
    elif dist == "outlier_cols":
        x[:, torch.randperm(D, generator=gen, device="cuda")[:int(round(0.01 * D))]] *= 20.0
    elif dist == "normal_2_3":
        x = 2.0 + math.sqrt(3.0) * x
    return x.to(torch.bfloat16)


def _normal(gen, rows, cols, std):
    return torch.randn(rows, cols, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(std)


def _uniform(gen, n):
    return (0.5 + torch.rand(n, generator=gen, device="cuda")).to(torch.bfloat16)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    bf = dict(device="cuda", dtype=torch.bfloat16)
    s = {"case": case}
    if case["op"] == "ffn":
        M, D, F = case["M"], case["D"], case["F"]
        s["X"] = _draw_x(gen, M, D, case["x"])
        s["g"] = _uniform(gen, D)
        up, down = ((F, D), (D, F)) if case["transposed"] else ((D, F), (F, D))
        s["W1"] = _normal(gen, *up, 1 / math.sqrt(D))
        s["W3"] = _normal(gen, *up, 1 / math.sqrt(D))
        s["W2"] = _normal(gen, *down, 1 / math.sqrt(F))
        s["Y"] = torch.empty(M, D, **bf)
    elif case["op"] == "ln":
        M, D, N = case["M"], case["D"], case["N"]
        s["X"] = _draw_x(gen, M, D, "normal_2_3")
        s["gamma"] = _uniform(gen, D)
        s["beta"] = (math.sqrt(0.1) * torch.randn(D, generator=gen, device="cuda")).to(torch.bfloat16)
        s["W"] = _normal(gen, *((N, D) if case["transposed"] else (D, N)), 1 / math.sqrt(D))
        s["Y"] = torch.empty(M, N, **bf)
    else:
        B, M, N, d, dv = (case[k] for k in ("B", "M", "N", "d", "dv"))
        for name, shape in (("Q", (B, M, d)), ("K", (B, N, d)), ("V", (B, N, dv))):
            s[name] = torch.randn(*shape, generator=gen, **bf)
        s["O"] = torch.empty(B, M, dv, **bf)
    return s


def run(s):
    c = s["case"]
    if c["op"] == "ffn":
        if c["residual"]:       # y = x + FFN(norm(x)), the block's own input as the residual
            return bb.bb_rmsnorm_swiglu_ffn_residual(s["X"], s["g"], s["W1"], s["W3"], s["W2"], s["X"], c["eps"],
                                                     Y=s["Y"], transposed=c["transposed"])
        fn = bb.bb_rmsnorm_swiglu_ffn_t if c["transposed"] else bb.bb_rmsnorm_swiglu_ffn
        return fn(s["X"], s["g"], s["W1"], s["W3"], s["W2"], c["eps"], Y=s["Y"])
    if c["op"] == "ln":
        fn = bb.bb_layernorm_matmul_t if c["transposed"] else bb.bb_layernorm_matmul
        return fn(s["X"], s["gamma"], s["beta"], s["W"], c["eps"], Y=s["Y"])
    return bb.bb_attention(s["Q"], s["K"], s["V"], O=s["O"])


def work(case):
    """bytes: every operand once, bf16; flops: the matrix products"""
    if case["op"] == "ffn":
        M, D, F = case["M"], case["D"], case["F"]
        return {"bytes": 2 * (3 * D * F + 2 * M * D + D), "flops": 6 * M * D * F}
    if case["op"] == "ln":
        M, D, N = case["M"], case["D"], case["N"]
        return {"bytes": 2 * (D * N + M * D + M * N + 2 * D), "flops": 2 * M * D * N}
    B, M, N, d, dv = (case[k] for k in ("B", "M", "N", "d", "dv"))
    return {"bytes": 2 * B * (M * (d + dv) + N * (d + dv)), "flops": 2 * B * M * N * (d + dv)}


def tolerance(case):
    """bf16 operands, intermediates and results around fp32 sums; each about four times what the operators show
    against the same operators in 64 bits (see TOLERANCES)"""
    rel, peak = TOLERANCES[case["op"]]
    return {"rel": rel, "max": peak}


# measured over the listed and drawn cases, relative and largest: ffn 3.4e-3 and 1.9e-2, ln 3.1e-3 and 1.8e-2,
# attention 2.4e-3 and 1.2e-2
TOLERANCES = {"ffn": (1.4e-2, 0.08), "ln": (1.2e-2, 0.07), "attention": (1e-2, 0.05)}
