"""The work that programs have this library do, as cases that can be timed: one chunk's hand-over between the model
and the KV cache, one chunk's forward or backward, a whole attention layer under Alg. 1 / Alg. 2 in either backward
order, and a training step of a small decoder.  Sizes are those of `workloads.CONFIGS` and of the tests, and the
ranges between and around them.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program holds before the call (tensors on the GPU)
    run(state)          one pass through the public entry points; returns everything it computes
    work(case)          bytes and floating-point operations that a pass cannot do without
    tolerance(case)     how far two correct implementations of the same precision may differ
"""
import torch

import paper_2505_16710_amd as seco
from paper_2505_16710_amd.chunk_loop import ChunkedDecoder

DEV = "cuda:0"
ROPE_BASE = 500000.0
_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, **kw):
    c = {"kind": kind, "dtype": "bf16", "batch": 1, "q_heads": 32, "kv_heads": 8, "head_dim": 128}
    c.update(kw)
    return {"name": name, **c} if name else c


def listed():
    return [
        # Between the projections and the attention of one layer: the shortest chunk of the paper's chunk-size study
        # at the end of its 16K-token context (a call of a few microseconds), and a 2048-token chunk at 32K tokens.
        _case("handover_c32", "handover", chunk=32, q_start=16352, rope=True),
        _case("handover_c2048", "handover", chunk=2048, q_start=30720, rope=True),
        # Forward: the shortest chunk against a long cache (a ragged tail, inference); a chunk length and position
        # that fit no tile; the whole sequence in one call (stage 1 run as a plain prefill).
        _case("fwd_c32_16k", "forward", chunk=32, q_start=16352),
        _case("fwd_ragged_c1000", "forward", chunk=1000, q_start=13777),
        _case("prefill_16k", "forward", chunk=16384, q_start=0),
        # Backward of one chunk: the paper's chunk length at 16K tokens; two sequences with ragged sizes; a selected
        # chunk of SpaCO (4 of 16 chunks of a 32K-token layer).
        _case("bwd_c128_16k", "backward", chunk=128, q_start=16256, t=0, sparse_dq=False),
        _case("bwd_ragged_c777_b2", "backward", batch=2, chunk=777, q_start=9324, t=0, sparse_dq=False),
        _case("spaco_bwd_c2048_32k", "backward", chunk=2048, q_start=30720, t=4, sparse_dq=False),
        # Second loop of Alg. 1 over a layer: the benchmark's headline (32K tokens, chunks of 2048); the 16K-token
        # layer in the transposed backward order; the fp32 configuration.
        _case("layer_32k_c2048", "layer", tokens=32768, chunk=2048, t=0, transposed=False),
        _case("layer_16k_c1024_transposed", "layer", tokens=16384, chunk=1024, t=0, transposed=True),
        _case("layer_f32_1k", "layer", dtype="f32", q_heads=4, kv_heads=4, head_dim=64, tokens=1024, chunk=256, t=0,
              transposed=False),
        # A whole training step (both loops of Alg. 1, two decoder layers, rotary embedding) as chunk_loop drives it.
        _case("train_4k_c512", "train", q_heads=8, kv_heads=2, tokens=4096, chunk=512, t=0, d_model=1024, layers=2),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choice(("handover", "forward", "forward", "backward", "backward", "backward", "layer", "layer", "f32",
                       "train"))
    hq, hkv = rng.choice(((32, 8), (32, 8), (32, 8), (16, 8), (16, 2), (8, 8)))
    heads = {"batch": rng.choice((1, 1, 2)), "q_heads": hq, "kv_heads": hkv}
    if kind == "handover":
        chunk = _log(rng, 16, 4096)
        return _case(None, kind, chunk=chunk, q_start=_log(rng, 1, 32768), rope=rng.random() < 0.6,
                     dtype=rng.choice(("bf16", "bf16", "bf16", "f32")), **heads)
    if kind == "forward":
        chunk = _log(rng, 1, 8192)
        return _case(None, kind, chunk=chunk, q_start=rng.choice((0, _log(rng, 256, 32768), _log(rng, 4096, 32768))),
                     **heads)
    if kind == "backward":
        chunk = _log(rng, 16, 4096)
        k = max(2, min(64, _log(rng, 1024, 32768) // chunk))       # chunks up to and including this one
        t = rng.choice((0, 0, min(k, 2), min(k, 4), min(k, 8)))
        q_start = (k - 1) * chunk if t else _log(rng, 1, 32768)
        return _case(None, kind, chunk=chunk, q_start=q_start, t=t, sparse_dq=bool(t) and rng.random() < 0.4, **heads)
    if kind == "layer":
        tokens = _log(rng, 2048, 16384)
        chunk = 64 * _log(rng, max(1, tokens // 64 // 48), max(2, tokens // 128))   # at most about 48 chunks
        tokens += rng.choice((0, rng.randrange(1, chunk)))                          # the last chunk may be short
        t = rng.choice((0, 0, min(4, -(-tokens // chunk))))
        return _case(None, kind, tokens=tokens, chunk=chunk, t=t, transposed=rng.random() < 0.25, **heads)
    if kind == "f32":
        tokens = _log(rng, 200, 1500)
        hq, hkv = rng.choice(((4, 4), (4, 2), (3, 3)))
        return _case(None, "layer", dtype="f32", batch=1, q_heads=hq, kv_heads=hkv, head_dim=rng.choice((32, 64, 80, 128)),
                     tokens=tokens, chunk=_log(rng, 64, 512), t=rng.choice((0, 0, 2)) if tokens > 1024 else 0,
                     transposed=False)
    tokens = 64 * _log(rng, 16, 64)
    chunk = 64 * -(-(tokens // 64) // rng.randrange(2, 9))                          # two to eight chunks
    return _case(None, "train", q_heads=8, kv_heads=2, tokens=tokens, chunk=chunk,
                 t=rng.choice((0, 0, min(2, -(-tokens // chunk)))), d_model=1024, layers=2)


def _spaced(k, t):
    """t of k chunks, evenly spaced, the last one among them; descending."""
    return sorted({k - 1 - i * k // t for i in range(t)}, reverse=True)


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    c, dt = case, _DTYPES[case["dtype"]]
    B, Hq, Hkv, D = c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"]

    def normal(*shape, dtype=dt):
        return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32).to(dtype)

    def projected(H, rows):     # as a projection leaves it: [B, rows, H, D] seen as [B, H, rows, D]
        return normal(B, rows, H, D).transpose(1, 2)

    s = {"case": case, "scale": D ** -0.5}
    if c["kind"] == "handover":
        C, N = c["chunk"], c["q_start"] + c["chunk"]
        s.update(k_new=projected(Hkv, C), v_new=projected(Hkv, C), k=normal(B, Hkv, N, D), v=normal(B, Hkv, N, D),
                 gk=normal(B, Hkv, N, D, dtype=torch.float32), gv=normal(B, Hkv, N, D, dtype=torch.float32))
        if c["rope"]:
            s.update(q=normal(B, Hq, C, D), dq=normal(B, Hq, C, D))
        else:
            s.update(gk2=normal(B, Hkv, N, D, dtype=torch.float32), gv2=normal(B, Hkv, N, D, dtype=torch.float32))
        return s
    if c["kind"] in ("forward", "backward"):
        C, N = c["chunk"], c["q_start"] + c["chunk"]
        s.update(q=normal(B, Hq, C, D), k=normal(B, Hkv, N, D), v=normal(B, Hkv, N, D))
        if c["kind"] == "backward":
            s["do"] = normal(B, Hq, C, D)
            s["o"], s["lse"] = seco.seco_chunk_attn_fwd(s["q"], s["k"], s["v"], c["q_start"], s["scale"])
            s["gk"], s["gv"] = (torch.zeros(B, Hkv, N, D, device=DEV) for _ in range(2))
            if c["t"]:
                k, t = N // C, c["t"]
                sel = _spaced(k, t)
                s["w"] = seco.spaco_chunk_weights(sel, k - 1, seco.spaco_compensation_factor(k, t))
                if c["sparse_dq"]:
                    f = (k - 1) / (t - 1) if t > 1 else 1.0
                    s["wq"] = [f if i in sel else 0.0 for i in range(k - 1)] + [1.0]
        return s
    if c["kind"] == "layer":
        N, C = c["tokens"], c["chunk"]
        k = -(-N // C)
        s.update(q=normal(B, Hq, N, D), k=normal(B, Hkv, N, D), v=normal(B, Hkv, N, D), do=normal(B, Hq, N, D))
        s["o"], s["dq"] = torch.zeros_like(s["q"]), torch.zeros_like(s["q"])
        s["gk"], s["gv"] = (torch.empty(B, Hkv, N, D, device=DEV) for _ in range(2))
        rows = (C + 3) // 4 * 4
        s["lse_all"] = torch.zeros(k, B * Hq * rows, device=DEV)
        s["lse"] = [s["lse_all"][j][:B * Hq * min(C, N - j * C)].view(B, Hq, -1) for j in range(k)]
        s["order"] = _spaced(k, c["t"]) if c["t"] else list(range(k - 1, -1, -1))
        s["factor"] = seco.spaco_compensation_factor(k, c["t"]) if c["t"] else 1.0
        if c["transposed"]:
            s["stats"] = torch.zeros(2, B, Hq, (N + 3) // 4 * 4, device=DEV)
        return s
    # train
    dm, vocab, ff = c["d_model"], 1024, 4 * c["d_model"]
    shapes = {"emb": (vocab, dm), "head": (dm, vocab), "norm_f": (dm,)}
    for i in range(c["layers"]):
        shapes.update({f"l{i}.norm1": (dm,), f"l{i}.norm2": (dm,), f"l{i}.wq": (dm, Hq * D), f"l{i}.wk": (dm, Hkv * D),
                       f"l{i}.wv": (dm, Hkv * D), f"l{i}.wo": (Hq * D, dm), f"l{i}.w1": (dm, ff), f"l{i}.w2": (ff, dm)})
    params = {}
    for n, sh in shapes.items():
        if len(sh) == 1:
            p = torch.ones(sh, device=DEV)
        else:
            p = torch.randn(sh, generator=gen, device=DEV) * (1.0 if n == "emb" else sh[0] ** -0.5)
        params[n] = p.to(dt).requires_grad_()
    s["decoder"] = ChunkedDecoder(params, c["layers"], Hq, Hkv, D, rope_base=ROPE_BASE)
    s["tokens"], s["targets"] = (torch.randint(0, vocab, (B, c["tokens"]), generator=gen, device=DEV) for _ in range(2))
    k = -(-c["tokens"] // c["chunk"])
    s["selected"] = _spaced(k, c["t"]) if c["t"] else None
    s["factor"] = seco.spaco_compensation_factor(k, c["t"]) if c["t"] else 1.0
    return s


def run(s):
    c, scale = s["case"], s["scale"]
    kind = c["kind"]
    if kind == "handover":
        C, s0, dt = c["chunk"], c["q_start"], s["k"].dtype
        if c["rope"]:
            q = seco.rope_rotate(s["q"], s0, ROPE_BASE)
            seco.kv_append(s["k_new"], s["v_new"], s["k"], s["v"], s0, rope_base=ROPE_BASE)
            dk, dv = seco.kvgrad_readout(s["gk"], s["gv"], s0, C, dt, rope_base=ROPE_BASE)
            dq = seco.rope_rotate(s["dq"], s0, ROPE_BASE, inverse=True)
            return {"q": q, "k": s["k"], "v": s["v"], "dk": dk, "dv": dv, "dq": dq}
        seco.kv_append(s["k_new"], s["v_new"], s["k"], s["v"], s0)
        seco.kvgrad_accumulate(s["gk"], s["gv"], s["gk2"], s["gv2"], 0.5, s0, s0 + C)     # the listing's relay
        dk, dv = seco.kvgrad_readout(s["gk"], s["gv"], s0, C, dt)
        return {"k": s["k"], "v": s["v"], "gk": s["gk"], "gv": s["gv"], "dk": dk, "dv": dv}
    if kind == "forward":
        o, lse = seco.seco_chunk_attn_fwd(s["q"], s["k"], s["v"], c["q_start"], scale)
        return {"o": o, "lse": lse}
    if kind == "backward":
        args = (s["q"], s["k"], s["v"], s["o"], s["lse"], s["do"], s["gk"], s["gv"], c["q_start"], scale)
        if c["t"]:
            dq = seco.spaco_chunk_attn_bwd(*args, s["w"], c["chunk"], dq_weight=s.get("wq"))
        else:
            dq = seco.seco_chunk_attn_bwd(*args)
        return {"dq": dq, "gk": s["gk"], "gv": s["gv"]}
    if kind == "layer":
        N, C, sel = c["tokens"], c["chunk"], s["order"]
        k = -(-N // C)
        seco.kvgrad_zero(s["gk"], s["gv"])
        for j in sel:
            s0 = j * C
            r = slice(s0, min(s0 + C, N))
            q, o, dq, lse = s["q"][:, :, r], s["o"][:, :, r], s["dq"][:, :, r], s["lse"][j]
            seco.seco_chunk_attn_fwd(q, s["k"], s["v"], s0, scale, o=o, lse=lse)
            if c["transposed"]:
                w = seco.spaco_gather_row_weights(sel, j, k, s["factor"]) if c["t"] else None
                seco.seco_chunk_attn_bwd_gather(s["q"][:, :, s0:], s["k"], s["v"], o, lse, s["do"][:, :, s0:], s["gk"],
                                                s["gv"], s0, scale, q.shape[2], s["stats"], d_q=dq, row_weight=w,
                                                weight_chunk_len=C if c["t"] else None)
            elif c["t"]:
                w = seco.spaco_chunk_weights(sel, j, s["factor"])
                seco.spaco_chunk_attn_bwd(q, s["k"], s["v"], o, lse, s["do"][:, :, r], s["gk"], s["gv"], s0, scale, w, C,
                                          d_q=dq)
            else:
                seco.seco_chunk_attn_bwd(q, s["k"], s["v"], o, lse, s["do"][:, :, r], s["gk"], s["gv"], s0, scale, d_q=dq)
        return {"o": s["o"], "lse": s["lse_all"], "dq": s["dq"], "gk": s["gk"], "gv": s["gv"]}
    loss, grads = s["decoder"].step(s["tokens"], s["targets"], c["chunk"], selected=s["selected"], factor=s["factor"])
    return {"loss": loss, **grads}


def _pairs(rows, q_start):
    return rows * q_start + rows * (rows + 1) // 2


def _fwd_bwd_flops(case):
    """Matrix work of the second loop over a layer, per unit of head_dim * query heads * batch."""
    N, C, t = case["tokens"], case["chunk"], case["t"]
    k = -(-N // C)
    sel = _spaced(k, t) if t else list(range(k))
    total = 0
    for j in sel:
        rows = min(C, N - j * C)
        seen = _pairs(rows, j * C)
        kept = rows * sum(C for i in sel if i < j) + rows * (rows + 1) // 2     # columns that receive dK/dV
        total += 4 * seen + 6 * seen + 4 * kept
    return total


def work(case):
    c = case
    B, Hq, Hkv, D = c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"]
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "handover":
        q, kv = B * Hq * c["chunk"] * D, B * Hkv * c["chunk"] * D
        if c["rope"]:
            return {"bytes": 2 * 2 * q * e + 2 * 2 * kv * e + 2 * kv * (4 + e), "flops": 3 * 2 * q + 3 * 2 * kv}
        return {"bytes": 2 * 2 * kv * e + 2 * 3 * kv * 4 + 2 * kv * e, "flops": 2 * 3 * kv}
    if c["kind"] == "forward":
        C, N = c["chunk"], c["q_start"] + c["chunk"]
        return {"bytes": B * (2 * Hq * C * D * e + Hq * C * 4 + 2 * Hkv * N * D * e),
                "flops": 4 * D * B * Hq * _pairs(C, c["q_start"])}
    if c["kind"] == "backward":
        C, N, t = c["chunk"], c["q_start"] + c["chunk"], c["t"]
        own = C * (C + 1) // 2
        seen, kept = _pairs(C, c["q_start"]), (t - 1) * C * C + own if t else _pairs(C, c["q_start"])
        g_rows, kv_rows = (t * C if t else N), (t * C if c["sparse_dq"] else N)
        return {"bytes": B * (4 * Hq * C * D * e + Hq * C * 4 + 2 * Hkv * kv_rows * D * e + 2 * 2 * Hkv * g_rows * D * 4),
                "flops": D * B * Hq * (6 * (kept if c["sparse_dq"] else seen) + 4 * kept)}
    if c["kind"] == "layer":
        N, C, t = c["tokens"], c["chunk"], c["t"]
        rows = min(N, t * C) if t else N
        return {"bytes": B * (4 * Hq * rows * D * e + Hq * rows * 4 + 2 * Hkv * N * D * e + 2 * Hkv * N * D * 4),
                "flops": D * B * Hq * _fwd_bwd_flops(c)}
    # train: every matrix once forward per loop and twice backward, attention as in "layer" plus the first loop
    N, C, dm = c["tokens"], c["chunk"], c["d_model"]
    k, t = -(-N // C), c["t"]
    weights = c["layers"] * (dm * (2 * Hq + 2 * Hkv) * D + 2 * dm * 4 * dm) + dm * 1024
    back = min(N, t * C) if t else N
    first = 4 * _pairs(N, 0) * D * Hq
    return {"bytes": 2 * (weights + 1024 * dm) * e,
            "flops": 2 * weights * (N + 3 * back) + c["layers"] * B * (first + D * Hq * _fwd_bwd_flops(c))}


def tolerance(case):
    if case["kind"] == "handover":
        # angles in fp64 and one rounding: results may differ where that rounding is a tie
        return {"rel": 1e-3 if case["dtype"] == "bf16" else 1e-6, "max": 1e-2 if case["dtype"] == "bf16" else 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    if case["kind"] == "train":
        return {"rel": 2e-2, "max": 0.5}     # two layers of bf16 activations and gradients around the kernels
    return {"rel": 1e-2, "max": 0.2}         # bf16 inputs, probabilities and results; fp32 sums
