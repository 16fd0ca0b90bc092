"""The work this library is used for, as cases to time: forwards of SVD-factored layers through the public binding.

A case is one pass of a user's program through ``SvdMlp`` (or, for callers that own their output and may not use the
workspace, ``svdmlp_forward_static_scratch``): ``layers`` gated MLP blocks or single factored layers of the same
extents, each with weights of its own, on ``M`` rows each.  The weights are laid out once in ``prepare`` (they are
constant at inference); a pass only runs forwards.

``listed`` holds the sizes that stand for each kind of use, ``draw`` more of the same ranges.
"""
import math

import torch

from paper_2510_25977_amd import binding as B

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, dtype, M, d, ffn, r, r_down=0, layers=1, static=False, outliers=False):
    c = dict(kind=kind, dtype=dtype, M=M, d=d, ffn=ffn, r=r, r_down=r_down, layers=layers, static=static, outliers=outliers)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest layer of the benchmark: one factored linear layer in fp32, two launches of next to no work
        _case("linear_f32_m32", "linear", "f32", 32, 256, 1024, 16),
        # a whole gated block in fp32, as someone does who checks a factorisation before going to bf16
        _case("gated_f32_m512", "gated", "f32", 512, 2048, 8192, 256, 256),
        # one token of one sequence through a stack of blocks: every forward reads weights nobody has touched lately
        _case("decode_m1", "gated", "bf16", 1, 4096, 14336, 512, 512, layers=8),
        # a batch of sequences, one token each, through the same stack
        _case("decode_m16", "gated", "bf16", 16, 4096, 14336, 512, 512, layers=8),
        # a single forward of a caller that cannot hand over per-call memory
        _case("decode_static_m4", "gated", "bf16", 4, 4096, 14336, 512, 512, static=True),
        # a larger decode batch at a rank that a mild compression keeps
        _case("batch_m64", "gated", "bf16", 64, 4096, 14336, 1024, 1024, layers=4),
        # the small layer of the benchmark, 128 rows
        _case("small_m128", "gated", "bf16", 128, 2048, 8192, 256, 256, layers=8),
        # a short prompt, an odd number of rows
        _case("prompt_m300", "gated", "bf16", 300, 4096, 14336, 512, 512),
        # extents off every tile: row count, intermediate width and both ranks odd, d a multiple of 128 only
        _case("ragged_m1777", "gated", "bf16", 1777, 2688, 7301, 331, 201),
        # the benchmark's headline prefill
        _case("prefill_m4096", "gated", "bf16", 4096, 4096, 14336, 512, 512),
        # the widest layer of the benchmark, with its power-law columns and outlier tokens
        _case("wide_m2048", "gated", "bf16", 2048, 5120, 27648, 1024, 1024, outliers=True),
        # the stand-alone factored layer at the shape of the paper's kernel evaluation
        _case("linear_m4096", "linear", "bf16", 4096, 8192, 16384, 4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _flops(c):
    if c["kind"] == "linear":
        return 2.0 * c["layers"] * c["M"] * c["r"] * (c["d"] + c["ffn"])
    return c["layers"] * c["M"] * (4.0 * c["r"] * (c["d"] + c["ffn"]) + 2.0 * c["r_down"] * (c["d"] + c["ffn"]))


def _factor_elements(c):
    if c["kind"] == "linear":
        return c["r"] * (c["d"] + c["ffn"])
    return (2 * c["r"] + c["r_down"]) * (c["d"] + c["ffn"])


_MOST_FLOPS = {"bf16": 8.0e11, "f32": 8.0e9}   # the largest listed case of the type
_MOST_FACTORS = 2.4e8                           # elements of one layer's factors


def draw(rng):
    """One more case: its kind of use first, then extents spread over that use's range."""
    use = rng.choice(["decode", "decode", "batch", "prompt", "prefill", "prefill", "linear", "linear", "f32"])
    while True:
        kind, dtype, static, outliers = "gated", "bf16", False, rng.random() < 0.15
        if use == "decode":
            M, static = _log(rng, 1, 32), rng.random() < 0.25
        elif use == "batch":
            M = _log(rng, 33, 128)
        elif use == "prompt":
            M = _log(rng, 129, 1024)
        elif use == "prefill":
            M = _log(rng, 1025, 8192)
        elif use == "linear":
            kind, M = "linear", _log(rng, 1, 8192)
        else:
            kind, dtype, M = rng.choice(["linear", "gated"]), "f32", _log(rng, 1, 512)
        if use == "f32":
            d, ffn = _log(rng, 96, 2048), _log(rng, 256, 8192)
            r = max(8, int(min(d, ffn) * rng.uniform(0.05, 0.5)))
        else:
            d = 128 * _log(rng, 8, 64)
            ffn = int(d * rng.uniform(2.0, 4.0))
            if kind == "linear":
                ffn = ffn // 128 * 128            # the row length of the output
            elif rng.random() < 0.7:
                ffn = ffn // 256 * 256            # widths as model configurations have them
            r = int(d * math.exp(rng.uniform(math.log(0.06), math.log(0.75))))
            if rng.random() < 0.7:
                r = max(128, r // 128 * 128)      # block-aligned ranks
        r_down = 0 if kind == "linear" else r if rng.random() < 0.6 else max(8, int(r * rng.uniform(0.5, 1.0)))
        c = _case(None, kind, dtype, M, d, ffn, r, r_down, 1, static, outliers)
        if M <= 128 and dtype == "bf16" and not static:
            c["layers"] = max(1, min(8, int(_MOST_FACTORS / _factor_elements(c))))
        if static and 8.5 * 2 ** 20 + 2 * 32 * (2 * (r + 63) + ffn + 256 + r_down + 255) > 15.9 * 2 ** 20:
            continue
        if _flops(c) <= _MOST_FLOPS[dtype] and _factor_elements(c) <= _MOST_FACTORS:
            return c


def _layer(case, g):
    """One layer's context and the activation that reaches it.  Factors ~ N(0, 1 / fan-in) and X ~ N(0, 1), so that
    every intermediate is O(1); with outliers, U's columns fall off like i^-0.5 and one entry of X in a hundred is 20
    times larger."""
    dt = _DTYPES[case["dtype"]]
    M, d, ffn, r, rd = case["M"], case["d"], case["ffn"], case["r"], case["r_down"]

    def normal(rows, cols, std):
        return torch.randn(rows, cols, generator=g, device="cuda", dtype=torch.float32).mul_(std)

    def u_like(rows, cols):
        u = normal(rows, cols, rows ** -0.5)
        if case["outliers"]:
            u *= torch.arange(1, cols + 1, device="cuda", dtype=torch.float32) ** -0.5
        return u.to(dt)

    def v_like(rows, cols):
        return normal(rows, cols, rows ** -0.5).to(dt)

    X = normal(M, d, 1.0)
    if case["outliers"]:
        X = torch.where(torch.rand(M, d, generator=g, device="cuda") < 0.01, X * 20.0, X)
    X = X.to(dt)
    if case["kind"] == "linear":
        return B.SvdMlp(max_M=M, Ug=u_like(d, r), Vg=v_like(r, ffn), kind=B.SVDMLP_LINEAR, keep_factors=False), X
    return B.SvdMlp(max_M=M, Ug=u_like(d, r), Vg=v_like(r, ffn), Uu=u_like(d, r), Vu=v_like(r, ffn), Ud=u_like(ffn, rd),
                    Vd=v_like(rd, d), keep_factors=False), X


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    layers = [_layer(case, g) for _ in range(case["layers"])]
    Y = [torch.empty_like(X) for _, X in layers] if case["static"] else None
    return dict(layers=layers, Y=Y)


def run(state):
    if state["Y"] is None:
        return [mlp(X) for mlp, X in state["layers"]]
    stream = torch.cuda.current_stream().cuda_stream
    for (mlp, X), Y in zip(state["layers"], state["Y"]):
        B.svdmlp_forward_static_scratch(mlp.ctx, X.data_ptr(), X.shape[0], Y.data_ptr(), stream)
    return state["Y"]


def work(case):
    """Factors and activation in once, result out once; multiply-adds of the factored products as two operations."""
    size = 2 if case["dtype"] == "bf16" else 4
    out = case["ffn"] if case["kind"] == "linear" else case["d"]
    return {"bytes": float(size * case["layers"] * (_factor_elements(case) + case["M"] * (case["d"] + out))), "flops": _flops(case)}


def tolerance(case):
    """Against the same chain in 64 bits: bf16 2.4e-3 (linear) to 4.1e-3 (gated) relative, 1.0e-2 to 3.6e-2 largest;
    fp32 1.4e-7 to 5.6e-7 relative, 3.1e-6 largest."""
    return {"rel": 1e-2, "max": 0.15} if case["dtype"] == "bf16" else {"rel": 3e-6, "max": 2e-5}
