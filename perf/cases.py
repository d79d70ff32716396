"""The work that programs built on this framework have it do, as cases that can be timed and compared.

A case is a dict of sizes and options; `prepare` makes what a program holds before the call (weights, caches,
captured graphs), `run` is one pass through the public calls, `exact` the same result in 64 bits from plain torch.

  quantize   a matrix of the FP16 parent into both draft formats (done once per matrix when a model is loaded)
  linear     the projections of some decoder layers, and the LM head, at m activation rows with one weight kind: the
             weight-streaming part of a draft step (INT4, FP8) or of a verification pass (FP16), as a captured graph
  attention  bias, rotation, cache write and causal attention of a block of new rows, layer after layer, as a graph
  sample     the draws of a round and its accept call over one draft chain per sequence (T > 0, or T = 0: greedy)
  multi      the accept call over several draft chains per sequence
  decoder    the k draft passes and the verification pass of a round through the decoder, on given tokens, as a graph
  prefill    the prompts of a batch into the caches of both models
"""
from __future__ import annotations

import math

import torch

import paper_2609_21704_amd as sq
from paper_2609_21704_amd.configs import Config
from paper_2609_21704_amd.decoder import EPS, THETA, DecoderWeights, SpecDecoder

HD = 128  # head dimension

# Shapes of the workloads in configs.py.
_1P5B = dict(hidden=1536, inter=8960, q_heads=12, kv_heads=2, vocab=151936)
_7B = dict(hidden=3584, inter=18944, q_heads=28, kv_heads=4, vocab=151936)


def listed():
    return [
        # a model's gate|up matrix quantized for both drafts when it is loaded
        dict(name="quantize_7b_gate_up", kind="quantize", n=37888, k=3584),
        # the smallest launches: draft projections of a small model, one sequence
        dict(name="draft_int4_1p5b_m1", kind="linear", variant="int4", m=1, layers=6, head=False, out="f16", **_1P5B),
        # a draft step of one sequence on a 7B model, with its LM head
        dict(name="draft_int4_7b_m1", kind="linear", variant="int4", m=1, layers=2, head=True, out="f16", **_7B),
        # the first draft step of a batch of four: two rows for every sequence
        dict(name="draft_int4_7b_m8", kind="linear", variant="int4", m=8, layers=2, head=True, out="f32", **_7B),
        # a draft step of a batch of four with the FP8 draft
        dict(name="draft_fp8_7b_m4", kind="linear", variant="fp8", m=4, layers=2, head=True, out="f16", **_7B),
        # verification of four sequences with eight drafts each
        dict(name="verify_f16_7b_m36", kind="linear", variant="f16", m=36, layers=1, head=True, out="f32", **_7B),
        # verification blocks of four sequences over long caches
        dict(name="attention_4x8192", kind="attention", b=4, rows=9, q_heads=28, kv_heads=4, context=8192, layers=4),
        # the sampling of one sequence's round at temperature 1
        dict(name="sample_t1_b1_k4", kind="sample", b=1, k=4, vocab=151936, t=1.0, probs=False),
        # greedy decoding of a batch of four
        dict(name="sample_greedy_b4_k4", kind="sample", b=4, k=4, vocab=151936, t=0.0, probs=False),
        # acceptance over four chains of two sequences
        dict(name="multi_b2_c4_k4", kind="multi", b=2, c=4, k=4, vocab=151936, t=1.0),
        # the passes of one sequence's round on a 7B-shaped decoder, about a thousand cached positions
        dict(name="decoder_7b_b1_k4", kind="decoder", variant="int4", b=1, k=4, context=1000, layers=4, **_7B),
        # two prompts of different lengths into both models' caches
        dict(name="prefill_7b_b2_1001", kind="prefill", variant="int4", b=2, length=1001, layers=6, **_7B),
    ]


# ------------------------------------------------------------------- draws
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _model(rng, grain, hidden_max):
    """Sizes of a model whose row lengths are multiples of `grain`."""
    hidden = grain * _log(rng, 896 // grain, hidden_max // grain)
    kv = rng.choice([1, 2, 4, 8])
    group = max(1, round(hidden / HD / kv * rng.uniform(0.7, 1.1)))
    while kv * group > 64:
        group -= 1
    return dict(hidden=hidden, inter=grain * round(hidden * rng.uniform(2.5, 5.5) / grain), q_heads=kv * group,
                kv_heads=kv, vocab=_log(rng, 4000, 152064))


def draw(rng):
    kind = rng.choice(["quantize", "linear", "linear", "linear", "linear", "attention", "sample", "multi", "decoder",
                       "prefill"])
    if kind == "quantize":
        return dict(kind=kind, n=_log(rng, 500, 40000), k=128 * _log(rng, 7, 64))
    if kind == "linear":
        variant = rng.choice(["int4", "fp8", "f16"])
        case = dict(kind=kind, variant=variant, m=_log(rng, 1, 64), layers=1, head=rng.random() < 0.5,
                    out=rng.choice(["f16", "f32"]), **_model(rng, {"int4": 128, "fp8": 16, "f16": 8}[variant], 5120))
        if work(case)["bytes"] > 1.5e9:
            case["head"] = False
        return case
    if kind == "attention":
        kv = rng.choice([1, 2, 4, 8])
        rows = rng.choice([1, 2, _log(rng, 1, 16), _log(rng, 1, 64)])
        b = _log(rng, 1, 8)
        context = max(rows, _log(rng, 64, max(65, min(16384, 4 * 4 * 8192 // (b * kv)))))
        return dict(kind=kind, b=b, rows=rows, q_heads=kv * rng.choice([1, 3, 4, 5, 6, 7, 8]), kv_heads=kv,
                    context=context, layers=rng.choice([1, 2, 3]))
    if kind == "sample":
        t = rng.choice([0.0, 0.7, 1.0])
        return dict(kind=kind, b=_log(rng, 1, 8), k=rng.randint(1, 8), vocab=_log(rng, 1000, 152064), t=t,
                    probs=t > 0 and rng.random() < 0.3)
    if kind == "multi":
        case = dict(kind=kind, b=_log(rng, 1, 4), c=rng.randint(2, 8), k=rng.randint(1, 6),
                    vocab=_log(rng, 1000, 152064), t=rng.choice([0.0, 0.7, 1.0]))
        while case["b"] * case["c"] * (2 * case["k"] + 1) > 100:
            case["c"] = max(2, case["c"] - 1)
            case["b"] = max(1, case["b"] - 1)
            case["k"] = max(1, case["k"] - 1)
        return case
    sizes = _model(rng, 128, 3584)
    b = _log(rng, 1, 8)
    if kind == "decoder":
        return dict(kind=kind, variant=rng.choice(["int4", "fp8"]), b=b, k=rng.randint(1, 64 // b - 1 if b > 6 else 8),
                    context=_log(rng, 64, 4096), layers=rng.randint(1, 3), **sizes)
    return dict(kind=kind, variant=rng.choice(["int4", "fp8"]), b=b, length=_log(rng, 12, 1200), layers=rng.randint(1, 3),
                **sizes)


# ------------------------------------------------------------------ inputs
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, *ids):
    s = int(seed) & 0x7FFFFFFF
    for i in ids:
        s = (s * 1000003 + int(i) + 1) % (1 << 61)
    return torch.Generator(device=_dev()).manual_seed(s)


def _normal(shape, std, g, dtype=torch.float32):
    return torch.randn(shape, generator=g, device=_dev()).mul_(std).to(dtype)


def _u24(shape, g):
    return torch.randint(0, 1 << 24, shape, generator=g, device=_dev(), dtype=torch.int32)


def _tokens(shape, vocab, g):
    return torch.randint(0, vocab, shape, generator=g, device=_dev(), dtype=torch.int32)


def _graph(fn):
    """fn captured as a HIP graph, after a first run outside capture (the library's workspace gets its size there)."""
    fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    return g


def _mats(case):
    """(n, k) of the projections of a case, in the order they run; the LM head last."""
    h, i, q, kv = case["hidden"], case["inter"], case["q_heads"] * HD, case["kv_heads"] * HD
    mats = [(q + 2 * kv, h), (h, q), (2 * i, h), (h, i)] * case["layers"]
    return mats + ([(case["vocab"], h)] if case.get("head", True) else [])


def _linear_inputs(case, seed, j, n, k):
    g = _gen(seed, 1, j)
    return _normal((n, k), 0.02, g, torch.float16), _normal((case["m"], k), 1.0, g, torch.float16)


def _contexts(case):
    """Cached positions of every sequence with its block's rows among them: ragged, the longest first."""
    return [max(case["rows"], case["context"] - s * case["context"] // (3 * case["b"])) for s in range(case["b"])]


def _attention_inputs(case, seed, layer):
    b, rows, hq, hkv = case["b"], case["rows"], case["q_heads"], case["kv_heads"]
    cap = -(-case["context"] // 64) * 64
    g = _gen(seed, 2, layer)
    return dict(qkv=_normal((b * rows, (hq + 2 * hkv) * HD), 1.2, g), bias=_normal(((hq + 2 * hkv) * HD,), 0.02, g, torch.float16),
                k=_normal((b, hkv, cap, HD), 1.2, g, torch.float16), v=_normal((b, hkv, HD, cap), 1.2, g, torch.float16))


def _sample_inputs(case, seed):
    b, k, v = case["b"], case["k"], case["vocab"]
    g = _gen(seed, 3)
    draft = _normal((k, b, v), 2.0, g)
    target = torch.cat([draft.permute(1, 0, 2) + _normal((b, k, v), 0.5, g), _normal((b, 1, v), 2.0, g)], 1)
    return dict(draft=draft, target=target.contiguous(), u_draft=_u24((k, b), g), u_accept=_u24((b, k + 1), g))


def _multi_inputs(case, seed):
    """Chains that share their first row, as their common context gives it, and diverge from there."""
    b, c, k, v = case["b"], case["c"], case["k"], case["vocab"]
    g = _gen(seed, 4)
    draft = _normal((k, b, c, v), 2.0, g)
    target = torch.empty((b, c, k + 1, v), device=_dev())
    draft[0] = draft[0, :, :1]
    for d in range(k):
        noise = _normal((b, c, v), 0.5, g)
        target[:, :, d] = draft[d] + (noise[:, :1] if d == 0 else noise)
    target[:, :, k] = _normal((b, c, v), 2.0, g)
    rows = torch.softmax(draft / max(case["t"], 0.5), -1).view(-1, v)
    tokens = torch.multinomial(rows, 1, generator=g).to(torch.int32).view(k, b, c)
    return dict(draft=draft, target=target, tokens=tokens, u=_u24((b, c * k + 1), g))


def _config(case, seed):
    return Config(0, "decoder", case["layers"], case["hidden"], case["inter"], case["q_heads"], case["kv_heads"],
                  case["vocab"], case["variant"], case.get("k", 4), case["b"], int(seed))


def _lengths(case):
    return [max(2, case["length"] - s * case["length"] // (3 * case["b"])) for s in range(case["b"])]


def _decoder_inputs(case, seed):
    """Positions, tokens and cache contents of a batch in the middle of its decoding."""
    b, k, v, layers, hkv = case["b"], case["k"], case["vocab"], case["layers"], case["kv_heads"]
    cap = -(-(case["context"] + k + 2) // 64) * 64
    g = _gen(seed, 5)
    ctx = [max(2, case["context"] - s * case["context"] // (3 * b)) for s in range(b)]
    s = dict(capacity=cap, pos=torch.tensor(ctx, dtype=torch.int32, device=_dev()), pending=_tokens((b,), v, g),
             prev=_tokens((b,), v, g), drafts=_tokens((k, b), v, g))
    for name in ("dk", "pk"):
        s[name] = _normal((layers, b, hkv, cap, HD), 1.2, g, torch.float16)
    for name in ("dv", "pv"):
        s[name] = _normal((layers, b, hkv, HD, cap), 1.2, g, torch.float16)
    return s


# ----------------------------------------------------------- prepare and run
def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return state["run"]()


def _prepare_quantize(case, seed):
    w = _normal((case["n"], case["k"]), 0.02, _gen(seed, 0), torch.float16)

    def run_():
        return [*sq.sq_quantize_int4_g128(w), *sq.sq_quantize_fp8_e4m3(w)]

    return {"run": run_}


def _prepare_linear(case, seed):
    variant, m = case["variant"], case["m"]
    out = {"f16": torch.float16, "f32": torch.float32}[case["out"]]
    mats, calls, ys = _mats(case), [], []
    for j, (n, k) in enumerate(mats):
        w, x = _linear_inputs(case, seed, j, n, k)
        y = torch.empty((m, n), dtype=torch.float32 if case["head"] and j == len(mats) - 1 else out, device=_dev())
        if variant == "int4":
            calls.append((sq.sq_qgemv_w4a16, (x, *sq.sq_quantize_int4_g128(w)), y))
        elif variant == "fp8":
            calls.append((sq.sq_qgemv_w8a16, (x, *sq.sq_quantize_fp8_e4m3(w)), y))
        else:
            calls.append((sq.sq_verify_gemm_f16, (x, w), y))
        ys.append(y)

    def step():
        for fn, args, y in calls:
            fn(*args, y=y)

    graph = _graph(step)

    def run_():
        graph.replay()
        return ys

    return {"run": run_, "calls": calls}


def _prepare_attention(case, seed):
    b, rows, hq, hkv = case["b"], case["rows"], case["q_heads"], case["kv_heads"]
    layers = [_attention_inputs(case, seed, l) for l in range(case["layers"])]
    pos = torch.tensor([c - rows for c in _contexts(case)], dtype=torch.int32, device=_dev())
    q = torch.empty((b * rows, hq, HD), dtype=torch.float16, device=_dev())
    outs = [torch.empty((b * rows, hq, HD), dtype=torch.float16, device=_dev()) for _ in layers]

    def step():
        for a, out in zip(layers, outs):
            if sq.sq_rope_attention_f16(a["qkv"], a["bias"], pos, 0, rows, hq, a["k"], a["v"], out, theta=THETA):
                continue
            sq.sq_rope_kv_f16(a["qkv"], a["bias"], pos, 0, rows, hq, a["k"], a["v"], theta=THETA, q_out=q)
            sq.sq_attention_f16(q, a["k"], a["v"], pos, 0, rows, out=out)

    graph = _graph(step)

    def run_():
        graph.replay()
        return [outs, [a["k"] for a in layers], [a["v"] for a in layers]]

    return {"run": run_, "inputs": (layers, pos, q)}


def _prepare_sample(case, seed):
    b, k, v, t = case["b"], case["k"], case["vocab"], case["t"]
    s = _sample_inputs(case, seed)
    i32 = dict(dtype=torch.int32, device=_dev())
    tokens, n_acc, nxt, none = (torch.empty(shape, **i32) for shape in ((k, b), (b,), (b,), (b,)))
    q_out = torch.empty_like(s["draft"]) if case["probs"] else None
    p_out = torch.empty_like(s["target"]) if case["probs"] else None

    def step():
        for i in range(k):
            sq.sq_spec_accept(None, s["draft"][i].view(b, 1, v), None, s["u_draft"][i].view(b, 1), t, n_accepted=none,
                              next_token=tokens[i])
        sq.sq_spec_accept(s["draft"], s["target"], tokens, s["u_accept"], t, n_accepted=n_acc, next_token=nxt,
                          q_out=q_out, p_out=p_out)

    graph = _graph(step)

    def run_():
        graph.replay()
        return [tokens, n_acc, nxt] + ([q_out, p_out] if case["probs"] else [])

    return {"run": run_, "inputs": (s, none)}


def _prepare_multi(case, seed):
    s = _multi_inputs(case, seed)
    outs = [torch.empty((case["b"],), dtype=torch.int32, device=_dev()) for _ in range(3)]

    def step():
        sq.sq_spec_accept_multi(s["draft"], s["target"], s["tokens"], s["u"], case["t"], n_accepted=outs[0],
                                next_token=outs[1], chain=outs[2])

    graph = _graph(step)

    def run_():
        graph.replay()
        return outs

    return {"run": run_, "inputs": s}


def _prepare_decoder(case, seed):
    b, k, v = case["b"], case["k"], case["vocab"]
    dec = SpecDecoder(DecoderWeights(_config(case, seed), _dev()), batch=b, k=k, capacity=_decoder_capacity(case))
    s = _decoder_inputs(case, seed)
    dec.dcache.k_all.copy_(s["dk"])
    dec.dcache.v_all.copy_(s["dv"])
    dec.pcache.k_all.copy_(s["pk"])
    dec.pcache.v_all.copy_(s["pv"])
    dec.pos_base.copy_(s["pos"])
    dec.pending.copy_(s["pending"])
    dec.prev.copy_(s["prev"])
    dec.draft_tokens.copy_(s["drafts"])

    def step():
        dec.forward(True, dec.prev, dec.pending.view(1, b), 2, -1, dec.draft_logits[0], last_only=True)
        for i in range(1, k):
            dec.forward(True, dec.draft_tokens[i - 1], None, 1, i, dec.draft_logits[i], last_only=True)
        dec.forward(False, dec.pending, dec.draft_tokens, k + 1, 0, dec.target_logits.view(b * (k + 1), v),
                    last_only=False)

    graph = _graph(step)

    def run_():
        graph.replay()
        return [dec.draft_logits, dec.target_logits, dec.dcache.k_all, dec.dcache.v_all, dec.pcache.k_all,
                dec.pcache.v_all]

    return {"run": run_, "decoder": dec}


def _decoder_capacity(case):
    return -(-(case["context"] + case["k"] + 2) // 64) * 64


def _prepare_prefill(case, seed):
    dec = SpecDecoder(DecoderWeights(_config(case, seed), _dev()), batch=case["b"], k=4,
                      capacity=-(-case["length"] // 64) * 64)
    prompt = _tokens((case["b"], case["length"]), case["vocab"], _gen(seed, 6)).cpu()
    lengths = _lengths(case)

    def run_():
        dec.prefill(prompt, lengths=lengths)
        return [dec.dcache.k_all, dec.dcache.v_all, dec.pcache.k_all, dec.pcache.v_all, dec.pos_base, dec.pending,
                dec.prev]

    return {"run": run_}


# -------------------------------------------------------------------- work
def _weight_bytes(variant, n, k):
    return n * k * 17 / 32 if variant == "int4" else (n * k + 4 * n if variant == "fp8" else 2 * n * k)


def work(case):
    kind = case["kind"]
    if kind == "quantize":  # each of the two calls reads the matrix
        nk = case["n"] * case["k"]
        return {"bytes": 4 * nk + nk * 17 / 32 + nk + 4 * case["n"], "flops": 6 * nk}
    if kind == "linear":
        m, mats = case["m"], _mats(case)
        total, flops = 0.0, 0.0
        for j, (n, k) in enumerate(mats):
            wide = case["out"] == "f32" or (case["head"] and j == len(mats) - 1)
            total += _weight_bytes(case["variant"], n, k) + 2 * m * k + (4 if wide else 2) * m * n
            flops += 2 * m * n * k
        return {"bytes": total, "flops": flops}
    if kind == "attention":
        rows, hq, hkv = case["rows"], case["q_heads"], case["kv_heads"]
        cached = sum(_contexts(case))
        new = case["b"] * rows
        return {"bytes": case["layers"] * (cached * hkv * HD * 4 + new * ((hq + 2 * hkv) * HD * 4 + hq * HD * 2 + hkv * HD * 4)),
                "flops": case["layers"] * cached * rows * hq * HD * 4}
    if kind == "sample":
        b, k, v = case["b"], case["k"], case["vocab"]
        rows = b * (2 * k + 1)
        return {"bytes": rows * v * (8 if case["probs"] else 4), "flops": rows * v * 4}
    if kind == "multi":
        rows = case["b"] * case["c"] * (2 * case["k"] + 1)
        return {"bytes": rows * case["vocab"] * 4, "flops": rows * case["vocab"] * 4}
    b, layers, hq, hkv = case["b"], case["layers"], case["q_heads"], case["kv_heads"]
    mats = _mats(dict(case, head=True))
    draft = sum(_weight_bytes(case["variant"], n, k) for n, k in mats)
    parent = sum(_weight_bytes("f16", n, k) for n, k in mats)
    params = sum(n * k for n, k in mats)
    if kind == "decoder":  # the passes follow one another: each reads its model's weights and the caches
        k = case["k"]
        cached = sum(max(2, case["context"] - s * case["context"] // (3 * b)) for s in range(b))
        rows = b * (k + 1)
        return {"bytes": k * draft + parent + (k + 1) * layers * cached * hkv * HD * 4 + (b * k + rows) * case["vocab"] * 4,
                "flops": 2 * params * (rows + b * (k + 1)) + layers * cached * hq * HD * 4 * (2 * k + 2)}
    n = b * (case["length"] - 1)  # no logits are asked for
    head = mats[-1][0] * mats[-1][1]
    return {"bytes": draft - _weight_bytes(case["variant"], *mats[-1]) + parent - _weight_bytes("f16", *mats[-1]) +
            2 * layers * n * hkv * HD * 4,
            "flops": 4 * (params - head) * n + 2 * layers * n * case["length"] / 2 * hq * HD * 4}


def tolerance(case):
    kind = case["kind"]
    if kind in ("quantize", "multi"):
        return "exact"
    if kind == "sample":  # tokens, and fp32 probabilities from 64-bit sums
        return {"rel": 1e-6} if case["probs"] else "exact"
    if kind == "linear":  # fp16 results round to 2^-11; fp32 ones differ by the order of their sums
        return {"rel": 1e-3} if case["out"] == "f16" else {"rel": 2e-6}
    if kind == "attention":  # fp16 queries, keys and results
        return {"rel": 1.5e-3}
    return {"rel": 5e-3}  # several layers, fp16 activations between them


# ------------------------------------------------------------------- exact
def _pow2(e):
    """2^e exactly, for integers e of a normal result."""
    return ((e.to(torch.int64) + 1023) << 52).view(torch.float64)


def _int4(w):
    """The values that the INT4 copy of w stands for, and its scales and zeros, in 64 bits."""
    n, k = w.shape
    v = w.double().view(n, k // 128, 128)
    lo, hi = v.amin(-1).clamp(max=0), v.amax(-1).clamp(min=0)
    s = (hi - lo) / 15
    sp = torch.clamp(torch.frexp(s)[1] - 1, min=-14) - 10
    s = torch.ceil(s * _pow2(-sp)) * _pow2(sp)
    none = hi == lo
    s = torch.where(none, torch.ones_like(s), s)
    z = torch.where(none, torch.zeros_like(s), torch.round(-lo / s).clamp(0, 15))
    q = (torch.round(v / s[..., None]) + z[..., None]).clamp(0, 15)
    return ((q - z[..., None]) * s[..., None]).view(n, k), s, z


def _fp8(w):
    """The values that the FP8 copy of w stands for, and its scales, in 64 bits."""
    amax = w.abs().amax(1).double()
    s = torch.where(amax == 0, torch.ones_like(amax), (amax / 448).float().double())
    t = w.double() / s[:, None]
    e = (torch.frexp(t)[1] - 1).clamp(min=-6)
    step = _pow2(e - 3)
    return torch.round(t / step).mul_(step).clamp_(-448, 448) * s[:, None], s


def _deq(variant, w):
    return _int4(w)[0] if variant == "int4" else (_fp8(w)[0] if variant == "fp8" else w.double())


def _mul(variant, x, w, rows=16384):
    """x . W'^T in 64 bits, some rows of W' at a time."""
    return torch.cat([x.double() @ _deq(variant, w[r:r + rows]).t() for r in range(0, w.shape[0], rows)], 1)


def _rope(u, pos):
    """u [rows][heads][128] turned to positions pos [rows]."""
    t = torch.arange(HD // 2, device=u.device, dtype=torch.float64)
    ang = pos.double()[:, None] * THETA ** (-2 * t / HD)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, e = u[..., :64], u[..., 64:]
    return torch.cat([a * c - e * s, e * c + a * s], -1)


def _attend(q, k, v, pos):
    """q [rows][hq][128] at positions pos over k, v [hkv][keys][128]."""
    rows, hq, _ = q.shape
    hkv = k.shape[0]
    s = torch.matmul(q.view(rows, hkv, hq // hkv, HD).permute(1, 2, 0, 3), k[:, None].transpose(-1, -2)) / math.sqrt(HD)
    keys = torch.arange(k.shape[1], device=q.device)
    s = s.masked_fill(keys[None, :] > pos[:, None], -math.inf)
    return torch.matmul(torch.softmax(s, -1), v[:, None]).permute(2, 0, 1, 3).reshape(rows, hq, HD)


def _block(qkv, bias, pos, hq, hkv, kc, vc):
    """One sequence's block: its rows' entries go into kc [hkv][cap][128], vc [hkv][128][cap] (64 bits); the attention."""
    u = (qkv.double() + bias.double()).view(qkv.shape[0], hq + 2 * hkv, HD)
    q, k, v = _rope(u[:, :hq], pos), _rope(u[:, hq:hq + hkv], pos), u[:, hq + hkv:]
    kc[:, pos] = k.transpose(0, 1)
    vc[:, :, pos] = v.permute(1, 2, 0)
    end = int(pos[-1]) + 1
    return _attend(q, kc[:, :end], vc[:, :, :end].transpose(1, 2), pos)


def _norm(h, w):
    return h / (h.square().mean(-1, keepdim=True) + EPS).sqrt() * w.double()


def _pass(weights, variant, tokens, pos, kc, vc):
    """All layers over one sequence's tokens at positions pos; the caches are [layers][hkv][...]; the last hidden rows."""
    cfg, st = weights.cfg, weights.stack
    h = weights.embed[tokens.long()].double()
    for l in range(weights.layers):
        qkv = _mul(variant, _norm(h, weights.in_norm[l]), st.w16[(l, "qkv")])
        a = _block(qkv, weights.qkv_bias[l], pos, cfg.q_heads, cfg.kv_heads, kc[l], vc[l])
        h = h + _mul(variant, a.reshape(len(tokens), -1), st.w16[(l, "o")])
        gu = _mul(variant, _norm(h, weights.post_norm[l]), st.w16[(l, "gate_up")])
        g, u = gu.chunk(2, -1)
        h = h + _mul(variant, g * torch.sigmoid(g) * u, st.w16[(l, "down")])
    return h


def exact(case, seed):
    kind = case["kind"]
    dev = _dev()
    if kind == "quantize":
        w = _normal((case["n"], case["k"]), 0.02, _gen(seed, 0), torch.float16)
        _, s4, z4 = _int4(w)
        return [None, s4, z4, None, _fp8(w)[1]]
    if kind == "linear":
        outs = []
        for j, (n, k) in enumerate(_mats(case)):
            w, x = _linear_inputs(case, seed, j, n, k)
            outs.append(_mul(case["variant"], x, w))
        return outs
    if kind == "attention":
        b, rows, hq, hkv = case["b"], case["rows"], case["q_heads"], case["kv_heads"]
        outs, ks, vs = [], [], []
        for l in range(case["layers"]):
            a = _attention_inputs(case, seed, l)
            kc, vc, out = a["k"].double(), a["v"].double(), []
            for s, c in enumerate(_contexts(case)):
                pos = torch.arange(c - rows, c, device=dev)
                out.append(_block(a["qkv"][s * rows:(s + 1) * rows], a["bias"], pos, hq, hkv, kc[s], vc[s]))
            outs.append(torch.cat(out))
            ks.append(kc)
            vs.append(vc)
        return [outs, ks, vs]
    if kind == "sample" and case["probs"]:
        s = _sample_inputs(case, seed)
        return [None, None, None, torch.softmax(s["draft"].double() / case["t"], -1),
                torch.softmax(s["target"].double() / case["t"], -1)]
    if kind == "decoder":
        w = DecoderWeights(_config(case, seed), dev)
        b, k = case["b"], case["k"]
        s = _decoder_inputs(case, seed)
        caches = {name: s[name].double() for name in ("dk", "dv", "pk", "pv")}
        head = w.stack.w16[(w.cfg.layers, "lm_head")]
        draft = torch.empty((k, b, case["vocab"]), dtype=torch.float64, device=dev)
        target = torch.empty((b, k + 1, case["vocab"]), dtype=torch.float64, device=dev)
        for r in range(b):
            p = int(s["pos"][r])
            toks = torch.cat([s["prev"][r:r + 1], s["pending"][r:r + 1], s["drafts"][:, r]])
            h = _pass(w, case["variant"], toks[:k + 1], torch.arange(p - 1, p + k, device=dev), caches["dk"][:, r],
                      caches["dv"][:, r])
            draft[:, r] = _mul(case["variant"], _norm(h[1:], w.final_norm), head)
            h = _pass(w, "f16", toks[1:], torch.arange(p, p + k + 1, device=dev), caches["pk"][:, r],
                      caches["pv"][:, r])
            target[r] = _mul("f16", _norm(h, w.final_norm), head)
        return [draft, target, caches["dk"], caches["dv"], caches["pk"], caches["pv"]]
    if kind == "prefill":
        w = DecoderWeights(_config(case, seed), dev)
        b, n, hkv, layers = case["b"], case["length"] - 1, case["kv_heads"], case["layers"]
        cap = -(-case["length"] // 64) * 64
        prompt = _tokens((b, case["length"]), case["vocab"], _gen(seed, 6))
        outs = []
        for variant in (case["variant"], "f16"):
            kc = torch.zeros((layers, b, hkv, cap, HD), dtype=torch.float64, device=dev)
            vc = torch.zeros((layers, b, hkv, HD, cap), dtype=torch.float64, device=dev)
            for r in range(b):
                _pass(w, variant, prompt[r, :n], torch.arange(n, device=dev), kc[:, r], vc[:, r])
            outs += [kc, vc]
        return outs + [None, None, None]
    return None
