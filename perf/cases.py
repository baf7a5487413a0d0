"""The work whose time is kept an eye on: passes of the FP8 linear layer as a training or serving program makes them,
through the public entry points, over the sizes, data types and options that they take.

A case's `kind` is one of
  fwd     one Linear forward: (producer and) 1x128 quantizer of the input, then the block-scaled GEMM.
            m, n, k   tokens, output and input width
            pre       "none", or what the quantizer is fused with: "rmsnorm" or "swiglu" (gate | up input)
            x         type of the input, "bf16" or "f32";  out: type of the output
            weights   "kept" (codes at hand: serving, or further micro-batches of one step) or "fresh" (the optimizer
                      has just changed them: the pass quantizes them first)
            cache     what is left for the backward pass: "none", "fp8" (the codes themselves) or "e5m6"
  bwd     its backward: dX = dY W on the transposed weight codes, and dW += dY^T X in FP32; the token-axis tiles of X
          come from `cache`: "bf16" X, the "fp8" codes re-tiled, or the "e5m6" codes
  moe     expert FFN forward of `experts` local experts of 256 (top-8 of `tokens` tokens): quantizer, grouped gate|up
          GEMM with SwiGLU and the cast in its epilogue, grouped down GEMM
  update  AdamW on the weights of one layer, and its new weight codes in both layouts
`scales` is "fp32" or "pow2" (power-of-two factors, applied by the matrix instruction).
"""
from __future__ import annotations

import random

import torch

import paper_2412_19437_amd as ds3

DEVICE = "cuda"
HIDDEN, DENSE_INTER, MOE_INTER, N_ROUTED, TOP_K = 7168, 18432, 2048, 256, 8
LARGEST = 4096 * DENSE_INTER * HIDDEN                    # m * n * k of the largest listed GEMM


def _fwd(m, n, k, pre="none", x="bf16", out="bf16", weights="kept", cache="none", scales="fp32"):
    return dict(kind="fwd", m=m, n=n, k=k, pre=pre, x=x, out=out, weights=weights, cache=cache, scales=scales)


def _bwd(m, n, k, cache="bf16", scales="fp32"):
    return dict(kind="bwd", m=m, n=n, k=k, cache=cache, scales=scales)


def _moe(tokens, experts=32, hidden=HIDDEN, inter=MOE_INTER, scales="fp32"):
    return dict(kind="moe", tokens=tokens, experts=experts, hidden=hidden, inter=inter, scales=scales)


def _update(n, k, scales="fp32"):
    return dict(kind="update", n=n, k=k, scales=scales)


def listed():
    return [
        # the smallest layer of the tests and the benchmark (FP32 input): launches and host work
        dict(_fwd(256, 512, 1024, x="f32", weights="fresh"), name="small_f32"),
        # a decode step of the dense FFN: few tokens, the weights' stream
        dict(_fwd(32, DENSE_INTER, HIDDEN), name="decode_ffn_up"),
        # a ragged micro-batch between the two: odd token count, an output width that is no multiple of any tile,
        # FP32 output, E5M6 cache
        dict(_fwd(1333, 3000, 1536, out="f32", cache="e5m6"), name="ragged_f32_out"),
        # the MLA projections at both ends: the narrow latent one behind its norm, and the wide one whose output dominates
        dict(_fwd(8192, 576, HIDDEN, pre="rmsnorm", cache="fp8"), name="mla_kv_a"),
        dict(_fwd(8192, 32768, 512, cache="fp8"), name="mla_kv_b"),
        # the dense FFN in training: up-projection right after an optimizer step, and down-projection behind SwiGLU with
        # power-of-two scales
        dict(_fwd(4096, DENSE_INTER, HIDDEN, weights="fresh", cache="fp8"), name="ffn_up"),
        dict(_fwd(4096, HIDDEN, DENSE_INTER, pre="swiglu", cache="fp8", scales="pow2"), name="ffn_down_pow2"),
        # backward of the up-projection, and of the narrower MLA query projection from the FP8 cache
        dict(_bwd(4096, DENSE_INTER, HIDDEN), name="ffn_up_bwd"),
        dict(_bwd(8192, 1536, HIDDEN, cache="fp8", scales="pow2"), name="mla_q_a_bwd_pow2"),
        # one GPU's share of the experts: a training batch, and a decode batch of about four rows an expert
        dict(_moe(8192), name="moe"),
        dict(_moe(128), name="moe_decode"),
        # the optimizer step of the largest layer
        dict(_update(DENSE_INTER, HIDDEN), name="ffn_update"),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread evenly over its logarithm."""
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


def draw(rng: random.Random):
    kind = rng.choices(["fwd", "bwd", "moe", "update"], [6, 3, 2, 1])[0]
    scales = rng.choice(["fp32", "fp32", "pow2"])
    if kind == "moe":
        return _moe(_log(rng, 32, 8192), rng.choice([8, 16, 32]), 128 * rng.randint(8, 56), 128 * rng.randint(4, 16), scales)
    while True:
        if kind == "update":
            n, k = _log(rng, 64, DENSE_INTER), 16 * _log(rng, 16, 1152)
            if n * k <= DENSE_INTER * HIDDEN:
                return _update(n, k, scales)
        elif kind == "bwd":
            m, n, k = 128 * _log(rng, 1, 64), 128 * _log(rng, 1, 144), 16 * _log(rng, 16, 1152)
            if m * n * k <= LARGEST and n * k <= DENSE_INTER * HIDDEN:
                return _bwd(m, n, k, rng.choice(["bf16", "fp8", "e5m6"]), scales)
        else:
            m, n, k = _log(rng, 1, 8192), _log(rng, 64, 32768), 128 * _log(rng, 1, 144)
            if rng.random() < 0.5:
                n = max(64, n // 64 * 64)
            pre = rng.choice(["none", "none", "rmsnorm", "swiglu"])
            x = rng.choice(["bf16", "bf16", "f32"]) if pre == "none" else "bf16"
            cache = rng.choice(["none", "fp8", "e5m6"]) if pre == "none" and x == "bf16" else rng.choice(["none", "fp8"])
            if m * n * k <= LARGEST and n * k <= DENSE_INTER * HIDDEN and not (pre == "rmsnorm" and k > 8192):
                return _fwd(m, n, k, pre, x, rng.choice(["bf16", "bf16", "f32"]), rng.choice(["kept", "fresh"]), cache, scales)


def _op(name, case):
    """The entry point `name` in its form for the case's kind of scales."""
    return getattr(ds3, name + ("_pow2" if case["scales"] == "pow2" else ""))


def _randn(gen, shape, std=1.0, dtype=torch.bfloat16):
    return torch.randn(shape, generator=gen, device=DEVICE).mul_(std).to(dtype)


def _activations(gen, m, k, dtype=torch.bfloat16):
    """N(0, 1) with one channel in a hundred 50 times as large: the outlier channels that fine-grained scales are for."""
    x = torch.randn((m, k), generator=gen, device=DEVICE)
    cols = torch.randperm(k, generator=gen, device=DEVICE)[: max(1, k // 100)]
    x[:, cols] *= 50.0
    return x.to(dtype)


def _group_offsets(seed, rows, experts):
    """Row offsets of the experts' groups: `rows` routed rows, loads that spread as sigmoid routing with a bias spreads
    them (a quarter of the mean either way and more; empty groups where there are few rows)."""
    rng = random.Random(seed)
    loads = [rng.lognormvariate(0.0, 0.3) for _ in range(experts)]
    sizes = [0] * experts
    for g in rng.choices(range(experts), loads, k=rows):
        sizes[g] += 1
    off = [0]
    for s in sizes:
        off.append(off[-1] + s)
    return torch.tensor(off, dtype=torch.int32, device=DEVICE)


def _moe_rows(case):
    return max(1, case["tokens"] * TOP_K * case["experts"] // N_ROUTED)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    kind, s = case["kind"], {"case": case}
    if kind == "moe":
        g, h, i, rows = case["experts"], case["hidden"], case["inter"], _moe_rows(case)
        s["x"] = _randn(gen, (rows, h))
        s["off"] = _group_offsets(seed, rows, g)
        # (gate and up rows of w13 interleaved in blocks of 128, as the fused epilogue takes them)
        q, sc = _op("ds3_quant_w_128x128", case)(_randn(gen, (g * 2 * i, h), 0.02))
        s["w13"] = q.view(g, 2 * i, h), sc.view(g, 2 * i // 128, h // 128)
        q, sc = _op("ds3_quant_w_128x128", case)(_randn(gen, (g * h, i), 0.02))
        s["w2"] = q.view(g, h, i), sc.view(g, h // 128, i // 128)
        return s
    n, k = case["n"], case["k"]
    if kind == "update":
        s["w"] = _randn(gen, n * k, 0.02, torch.float32)
        s["grad"] = _randn(gen, n * k, 1e-3, torch.float32)
        s["m"] = _randn(gen, n * k, 1e-4)
        s["v"] = _randn(gen, n * k, 1e-3).square()
        s["w_bf16"] = torch.empty((n, k), dtype=torch.bfloat16, device=DEVICE)
        s["step"] = 100
        return s
    m = case["m"]
    if kind == "bwd":
        s["dy"] = _randn(gen, (m, n), 0.01)
        _, _, s["wt"], s["swt"] = _op("ds3_quant_w_128x128_dual", case)(_randn(gen, (n, k), 0.02))
        x = _activations(gen, m, k)
        s["x"] = {"bf16": lambda t: t, "fp8": _op("ds3_quant_act_1x128", case), "e5m6": ds3.ds3_quant_act_1x128_e5m6}[case["cache"]](x)
        s["dw"] = torch.zeros((n, k), dtype=torch.float32, device=DEVICE)
        return s
    dtype = torch.float32 if case["x"] == "f32" else torch.bfloat16
    s["x"] = _randn(gen, (m, 2 * k), 2.0) if case["pre"] == "swiglu" else _activations(gen, m, k, dtype)
    if case["pre"] == "rmsnorm":
        s["gamma"] = 1.0 + 0.1 * torch.randn(k, generator=gen, device=DEVICE)
    w = _randn(gen, (n, k), 0.02, dtype)
    s["w"] = w if case["weights"] == "fresh" else _op("ds3_quant_w_128x128", case)(w)
    return s


def _run_fwd(s, case):
    if case["weights"] == "fresh":
        qw, sw = _op("ds3_quant_w_128x128", case)(s["w"])
    else:
        qw, sw = s["w"]
    if case["pre"] == "rmsnorm":
        q, sc = _op("ds3_rmsnorm_quant_1x128", case)(s["x"], s["gamma"], 1e-6)
    elif case["pre"] == "swiglu":
        q, sc = _op("ds3_swiglu_quant_1x128", case)(s["x"])
    else:
        q, sc = _op("ds3_quant_act_1x128", case)(s["x"])
    y = _op("ds3_gemm_fp8_bs", case)(q, sc, qw, sw, out_dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16)
    if case["cache"] == "fp8":
        return y, q, sc
    if case["cache"] == "e5m6":
        return y, ds3.ds3_quant_act_1x128_e5m6(s["x"])
    return y


def _run_bwd(s, case):
    quant_t, gemm = _op("ds3_quant_act_128x1", case), _op("ds3_gemm_fp8_bs", case)
    q, sc = _op("ds3_quant_act_1x128", case)(s["dy"])
    dx = gemm(q, sc, s["wt"], s["swt"])
    dyt, sdyt = quant_t(s["dy"])
    if case["cache"] == "fp8":
        xt, sxt = _op("ds3_retile_1x128_to_128x1", case)(*s["x"])
    else:
        xt, sxt = quant_t(s["x"] if case["cache"] == "bf16" else ds3.ds3_dequant_e5m6(*s["x"]))
    gemm(dyt, sdyt, xt, sxt, sb_mode=ds3.DS3_BSCALE_PER_ROW, c=s["dw"], accumulate=True)
    return dx, s["dw"]


def _run_moe(s, case):
    q, sc = _op("ds3_quant_act_1x128", case)(s["x"])
    q, sc = _op("ds3_grouped_gemm_swiglu_quant_fp8_bs", case)(q, sc, s["off"], *s["w13"])
    return _op("ds3_grouped_gemm_fp8_bs", case)(q, sc, s["off"], *s["w2"])


def _run_update(s, case):
    s["step"] += 1
    ds3.ds3_adamw_bf16_states(s["w"], s["grad"], s["m"], s["v"], 2.2e-4, 0.9, 0.95, 1e-8, 0.1, s["step"],
                              w_bf16=s["w_bf16"].view(-1))
    codes = _op("ds3_quant_w_128x128_dual", case)(s["w_bf16"])
    return s["w"], s["m"], s["v"], s["w_bf16"], codes


_RUN = {"fwd": _run_fwd, "bwd": _run_bwd, "moe": _run_moe, "update": _run_update}


def run(state):
    return _RUN[state["case"]["kind"]](state, state["case"])


def _factor(amax, case):
    """(stored scale, multiplier) of groups with these maxima, in FP32 as the format fixes it; power-of-two scales are
    rounded up."""
    amax = amax.float()
    if case["scales"] == "pow2":
        m, e = torch.frexp(amax / 448.0)
        s = torch.ldexp(torch.ones_like(amax), torch.where(m == 0.5, e - 1, e))
        r = 1.0 / s
    else:
        s, r = amax / 448.0, torch.full_like(amax, 448.0) / amax
    return torch.where(amax == 0, 1.0, s), torch.where(amax == 0, 0.0, r)


def _rounded(x, case, rows, cols):
    """`x` as its codes and scales hold it, in 64 bits: groups of rows x cols, E4M3 codes."""
    m, k = x.shape
    xp = torch.nn.functional.pad(x.float(), (0, -k % cols, 0, -m % rows))
    g = xp.view(xp.shape[0] // rows, rows, xp.shape[1] // cols, cols)
    s, r = _factor(g.abs().amax((1, 3), keepdim=True), case)
    return ((g * r).to(torch.float8_e4m3fn).double() * s.double()).view(xp.shape)[:m, :k]


def _decoded(q, s, rows):
    """Codes and scales (groups of rows x 128) in 64 bits."""
    q, s = q.contiguous().view(torch.float8_e4m3fn).double(), s.double()
    return q * s.repeat_interleave(rows, 0).repeat_interleave(128, 1)[: q.shape[0], : q.shape[1]]


def _silu_mul(h):
    g, u = h.double().chunk(2, 1)
    return (g * torch.sigmoid(g) * u).bfloat16()         # a BF16 tensor, whoever produces it


def _exact_bwd(s, case):
    dy = s["dy"]
    dx = _rounded(dy, case, 1, 128) @ _decoded(s["wt"], s["swt"], 128).t()
    if case["cache"] == "bf16":
        x = s["x"]
    elif case["cache"] == "fp8":
        x = _decoded(*s["x"], 1).float()                 # the re-tiled values are FP32 products
    else:
        q, sc = s["x"]
        b = q.int().view(q.shape[0], -1, 3)              # two 12-bit codes in three bytes: the upper bits of binary16
        c = torch.stack((b[..., 0] | (b[..., 1] & 15) << 8, b[..., 1] >> 4 | b[..., 2] << 4), -1).view(q.shape[0], -1)
        x = (c << 4).to(torch.int16).view(torch.float16).float() * sc.repeat_interleave(128, 1)[:, : c.shape[1]]
    return dx, _rounded(dy, case, 128, 1).t() @ _rounded(x, case, 128, 1)


def _exact_moe(s, case):
    h, i, y = case["hidden"], case["inter"], []
    off = s["off"].tolist()
    for e in range(case["experts"]):
        x = _rounded(s["x"][off[e] : off[e + 1]], case, 1, 128)
        gu = (x @ _decoded(s["w13"][0][e], s["w13"][1][e], 128).t()).bfloat16()
        gu = gu.view(-1, i // 128, 2, 128).transpose(1, 2).reshape(-1, 2 * i)
        y.append(_rounded(_silu_mul(gu), case, 1, 128) @ _decoded(s["w2"][0][e], s["w2"][1][e], 128).t())
    return torch.cat(y)


def _exact_update(s, case):
    w, g, m, v = (s[t].double() for t in ("w", "grad", "m", "v"))
    t = s["step"] + 1
    m, v = 0.9 * m + 0.1 * g, 0.95 * v + 0.05 * g * g
    w = w - 2.2e-4 * (m / (1 - 0.9**t) / ((v / (1 - 0.95**t)).sqrt() + 1e-8) + 0.1 * w)
    return w, m, v, w.view_as(s["w_bf16"]), None


def exact(case, seed):
    """What `run` returns, with the codes and scales as the formats fix them and every sum in 64 bits; no value for
    codes, whose bits are compared as they are."""
    s = prepare(case, seed)
    if case["kind"] != "fwd":
        return {"bwd": _exact_bwd, "moe": _exact_moe, "update": _exact_update}[case["kind"]](s, case)
    x = s["x"]
    if case["pre"] == "swiglu":
        x = _silu_mul(x)
    elif case["pre"] == "rmsnorm":
        x = x.double()
        x = (x * (x.square().mean(1, keepdim=True) + 1e-6).rsqrt() * s["gamma"].double()).bfloat16()
    w = _rounded(s["w"], case, 128, 128) if case["weights"] == "fresh" else _decoded(*s["w"], 128)
    y = _rounded(x, case, 1, 128) @ w.t()
    return {"none": y, "fp8": (y, None, None), "e5m6": (y, None)}[case["cache"]]


def _codes(rows, cols):
    """Bytes of 1x128-quantized codes and their scales."""
    return rows * cols + rows * ((cols + 127) // 128) * 4


def work(case):
    kind = case["kind"]
    if kind == "moe":
        rows, g, h, i = _moe_rows(case), case["experts"], case["hidden"], case["inter"]
        used = min(rows, g)                              # experts that can have rows at all
        return {"bytes": rows * h * 2 + used * 3 * i * h * (1 + 4 / 16384) + rows * h * 2, "flops": 6 * rows * i * h}
    n, k = case["n"], case["k"]
    if kind == "update":
        return {"bytes": n * k * (4 + 4 + 2 + 2 + 4 + 2 + 2 + 2 + 1 + 1), "flops": 15 * n * k}
    m = case["m"]
    if kind == "bwd":
        x = {"bf16": m * k * 2, "fp8": _codes(m, k), "e5m6": m * k * 3 // 2 + m * ((k + 127) // 128) * 4}[case["cache"]]
        return {"bytes": m * n * 2 + n * k + x + m * k * 2 + n * k * 8, "flops": 4 * m * n * k}
    es, os = 4 if case["x"] == "f32" else 2, 4 if case["out"] == "f32" else 2
    w = n * k * es if case["weights"] == "fresh" else n * k
    left = {"none": 0, "fp8": _codes(m, k), "e5m6": m * k * 3 // 2}[case["cache"]]
    return {"bytes": m * k * es * (2 if case["pre"] == "swiglu" else 1) + w + m * n * os + left, "flops": 2 * m * n * k}


def tolerance(case):
    """About four times what the path differs by from itself with the order of every sum changed (K permuted inside and
    across its blocks), measured over the listed and drawn cases; AdamW: from its FP64 form.  Codes and scales of a
    quantizer are exact, except behind a sum (RMSNorm: 1.2e-7 of the codes) and behind the optimizer."""
    kind = case["kind"]
    if kind == "moe":                                     # rel 2.9e-3: a BF16 activation an ulp off may move a code
        return {"rel": 8e-3, "max": 0.25}
    if kind == "update":                                  # the BF16 moments: rel 1.8e-5, one BF16 ulp at most
        return {"rel": 7e-5, "max": 0.03, "differ": 1e-6}
    if kind == "bwd":                                     # BF16 dX: rel 2.3e-4, one BF16 ulp at most
        return {"rel": 1e-3, "max": 0.03}
    differ = 1e-6 if case["pre"] == "rmsnorm" else 0.0
    if case["out"] == "f32":                              # rel 8.5e-5 (the matrix unit's own sum of 128 products)
        return {"rel": 3.5e-4, "max": 5e-3, "differ": differ}
    return {"rel": 2e-3, "max": 0.03, "differ": differ}   # BF16 output: rel 5.7e-4, one BF16 ulp at most
