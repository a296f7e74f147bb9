"""Performance cases: the calls a streaming video-DiT program makes of this package.

The shapes are those of the benchmark and the parity tests: a chunk of 3 latent
frames of 1560 tokens (4680 queries), 12 heads of 128 (hidden 1536, "1.3B") and
40 heads of 128 (hidden 5120, "14B"), the tiny parity shape (2 heads of 64), and
generic ones between them. Kinds:

  attn     one chunk's attention over a layer's cache: the warmup's dual-stream
           pass, an F-Layer (full cache) or an L-Layer (sink + window)
  accum    the warmup statistics of one chunk, from cleared statistics
  solve    the closed-form modulation of one layer at the end of warmup
  batch    the same for all layers at once
  project  the output projection of an L-Layer (bf16)
  w8a8     its W8A8 form: activations quantised, then the int8 product
  convert  an absorbed layer's first chunk as an L-Layer: weight update, eviction
           into the ring, append of the chunk, attention, projection
"""

import math

import torch

import paper_2607_00712_amd as ispa

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
DTYPES = {"bf16": BF16, "f32": F32}
LAM = 1e-3


def listed():
    return [
        # the parity tests' shape: all latency, head_dim 64, ends in two short key ranges
        {"name": "attn_tiny_dual", "kind": "attn", "heads": 2, "head_dim": 64, "n_q": 64, "cache_len": 256,
         "window": 64, "sink": 0, "dual": True},
        # streaming one latent frame at a time, 24 heads of 64, sink frame + three recent frames
        {"name": "attn_frame_d64", "kind": "attn", "heads": 24, "head_dim": 64, "n_q": 1560, "cache_len": 32760,
         "window": 4680, "sink": 1560, "dual": False},
        # an L-Layer's chunk at the 1.3B shape: what half of the layers do all through a rollout
        {"name": "attn_local_1p3b", "kind": "attn", "heads": 12, "head_dim": 128, "n_q": 4680, "cache_len": 32760,
         "window": 9360, "sink": 0, "dual": False},
        # the warmup's dual-stream pass at the 1.3B shape, full and local result in one call
        {"name": "attn_dual_1p3b", "kind": "attn", "heads": 12, "head_dim": 128, "n_q": 4680, "cache_len": 32760,
         "window": 9360, "sink": 0, "dual": True},
        # an F-Layer late in a video at the 14B shape: the largest call
        {"name": "attn_full_14b", "kind": "attn", "heads": 40, "head_dim": 128, "n_q": 4680, "cache_len": 98280,
         "window": 98280, "sink": 0, "dual": False},
        # one warmup chunk's statistics, fp32 attention outputs as they come from attention
        {"name": "accum_1p3b", "kind": "accum", "d_in": 1536, "d_out": 1536, "rows": 4680, "x": "f32", "y": "f32"},
        # one layer's solve, the caller waiting for its eps
        {"name": "solve_1p3b", "kind": "solve", "d_in": 1536, "d_out": 1536, "rows": 9360, "wait": True},
        # one layer's solve at the 14B shape, enqueued
        {"name": "solve_14b", "kind": "solve", "d_in": 5120, "d_out": 5120, "rows": 18720, "wait": False},
        # every layer's solve at the end of warmup
        {"name": "batch_1p3b", "kind": "batch", "layers": 30, "d_in": 1536, "d_out": 1536, "rows": 4680},
        # the output projection of a 14B chunk
        {"name": "project_14b", "kind": "project", "rows": 4680, "d_in": 5120, "d_out": 5120, "out": "bf16"},
        # the W8A8 projection of a 1.3B chunk with its activations' quantisation
        {"name": "w8a8_1p3b", "kind": "w8a8", "rows": 4680, "d_in": 1536, "d_out": 1536, "out": "bf16"},
        # a layer becomes an L-Layer and serves its first chunk
        {"name": "convert_1p3b", "kind": "convert", "heads": 12, "head_dim": 128, "n_q": 4680, "cache_len": 18720,
         "window": 9360, "sink": 0},
    ]


# a drawn case does at most the operations of the largest listed attention call
MOST_ATTN = 4 * 4680 * 98280 * 5120


def _log(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def _attn_shape(rng, heads_hi=40, n_q_hi=4680, keys_hi=98280):
    while True:
        head_dim = rng.choice((64, 128, 128))
        heads = rng.randint(1, heads_hi)
        n_q = _log(rng, 64, n_q_hi)
        n = max(n_q, _log(rng, 256, keys_hi))
        if 4 * n_q * n * heads * head_dim <= MOST_ATTN // 2:
            return heads, head_dim, n_q, n


def draw(rng):
    kind = rng.choice(("attn", "attn", "attn", "accum", "solve", "batch", "project", "w8a8", "convert"))
    if kind == "attn":
        heads, head_dim, n_q, n = _attn_shape(rng)
        window = max(n_q, _log(rng, 64, n))
        return {"kind": kind, "heads": heads, "head_dim": head_dim, "n_q": n_q, "cache_len": n, "window": window,
                "sink": rng.choice((0, 0, n_q, rng.randint(1, n))), "dual": rng.random() < 0.5}
    if kind == "accum":
        return {"kind": kind, "d_in": _log(rng, 128, 5120, 64), "d_out": _log(rng, 128, 5120, 8),
                "rows": _log(rng, 64, 4680), "x": rng.choice(("bf16", "f32")), "y": rng.choice(("bf16", "f32"))}
    if kind == "solve":
        d = _log(rng, 128, 4096, 64)
        return {"kind": kind, "d_in": d, "d_out": rng.choice((d, _log(rng, 128, 4096, 8))), "rows": 4 * d,
                "wait": rng.random() < 0.5}
    if kind == "batch":
        d = _log(rng, 128, 2048, 64)
        return {"kind": kind, "layers": rng.randint(2, 30), "d_in": d, "d_out": rng.choice((d, _log(rng, 128, 2048, 8))),
                "rows": 3 * d}
    if kind in ("project", "w8a8"):
        return {"kind": kind, "rows": _log(rng, 64, 4680), "d_in": _log(rng, 128, 5120, 64),
                "d_out": _log(rng, 128, 5120, rng.choice((8, 64, 256))), "out": rng.choice(("bf16", "f32"))}
    heads, head_dim, n_q, n = _attn_shape(rng, 24, 4680, 32760)
    return {"kind": "convert", "heads": heads, "head_dim": head_dim, "n_q": n_q, "cache_len": n,
            "window": max(n_q, _log(rng, 64, 9360)), "sink": rng.choice((0, min(n_q, n)))}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + 17)
    return g


def _randn(g, *shape, dtype=F32):
    return torch.randn(*shape, generator=g, device="cuda", dtype=F32).to(dtype)


def _warmup_rows(g, rows, d_in, d_out):
    """Statistics rows as a layer's attention gives them: channels of unequal
    scale, a discrepancy that the layer's input explains in part."""
    x = _randn(g, rows, d_in) * torch.logspace(0, -1, d_in, device="cuda")
    y_local = _randn(g, rows, d_out)
    w = _randn(g, d_in, d_out) * (1.0 / math.sqrt(d_in))
    y_full = y_local + x @ w + 0.1 * _randn(g, rows, d_out)
    return x, y_full, y_local


def _qkv(c, g, rows):
    hidden = c["heads"] * c["head_dim"]
    return (_randn(g, c["n_q"], hidden, dtype=BF16), _randn(g, rows, hidden, dtype=BF16),
            _randn(g, rows, hidden, dtype=BF16))


def _project_inputs(c, g):
    a = _randn(g, c["rows"], c["d_in"], dtype=BF16)
    w = (_randn(g, c["d_out"], c["d_in"]) * (1.0 / math.sqrt(c["d_in"]))).to(BF16)
    return a, w


def _convert_inputs(c, g):
    hidden = c["heads"] * c["head_dim"]
    q, k, v = _qkv(c, g, c["cache_len"])
    k_new, v_new = _randn(g, c["n_q"], hidden, dtype=BF16), _randn(g, c["n_q"], hidden, dtype=BF16)
    w0 = (_randn(g, hidden, hidden) * (1.0 / math.sqrt(hidden))).to(BF16)
    dw = _randn(g, hidden, hidden) * (0.1 / math.sqrt(hidden))
    return q, k, v, k_new, v_new, w0, dw


def _lower(G):
    """Views that cover the valid part of G, its lower triangle of 64 x 64
    blocks: diagonal blocks, the block left of every odd one, strips of 128 rows."""
    d = G.shape[0]
    n, base = d // 64, G.storage_offset()
    views = [G.as_strided((n, 64, 64), (64 * d + 64, d, 1), base)]
    if n > 1:
        views.append(G.as_strided((n // 2, 64, 64), (128 * d + 128, d, 1), base + 64 * d))
    return views + [G[a:min(a + 128, d), :a] for a in range(128, d, 128)]


def prepare(case, seed):
    c, g = case, _gen(seed)
    s = {"case": c}
    kind = c["kind"]
    if kind == "attn":
        s["q"], s["k"], s["v"] = _qkv(c, g, c["cache_len"])
    elif kind == "accum":
        x, y_full, y_local = _warmup_rows(g, c["rows"], c["d_in"], c["d_out"])
        s["x"], s["y_full"], s["y_local"] = x.to(DTYPES[c["x"]]), y_full.to(DTYPES[c["y"]]), y_local.to(DTYPES[c["y"]])
        s["stats"] = ispa.Stats(c["d_in"], c["d_out"])
        G, C, sq, _ = s["stats"].views()
        s["views"] = {"G": _lower(G), "C": C, "s": sq}
    elif kind == "solve":
        s["stats"] = ispa.Stats(c["d_in"], c["d_out"])
        s["stats"].accum(*_warmup_rows(g, c["rows"], c["d_in"], c["d_out"]))
        s["dw"] = torch.empty((c["d_in"], c["d_out"]), dtype=F32, device="cuda")
    elif kind == "batch":
        s["stats"] = ispa.StatsBatch(c["layers"], c["d_in"], c["d_out"])
        for layer in s["stats"].layers:
            layer.accum(*_warmup_rows(g, c["rows"], c["d_in"], c["d_out"]))
        s["dw"] = torch.empty((c["layers"], c["d_in"], c["d_out"]), dtype=F32, device="cuda")
    elif kind == "project":
        s["a"], s["w"] = _project_inputs(c, g)
    elif kind == "w8a8":
        s["a"], w = _project_inputs(c, g)
        s["q_w"], s["scale_w"] = ispa.quantize_rows(w)  # once, with the weights
    else:
        s["q"], s["k"], s["v"], s["k_new"], s["v_new"], s["w0"], s["dw"] = _convert_inputs(c, g)
        s["w"] = torch.empty_like(s["w0"])
        rows = min(c["sink"], c["cache_len"]) + c["window"]
        s["ring"] = tuple(torch.zeros((rows, c["heads"] * c["head_dim"]), dtype=BF16, device="cuda") for _ in "kv")
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "attn":
        return ispa.attn_chunk(s["q"], s["k"], s["v"], c["cache_len"], c["window"], c["heads"], sink_len=c["sink"],
                               dual=c["dual"])
    if kind == "accum":
        s["stats"].reset()
        s["stats"].accum(s["x"], s["y_full"], s["y_local"])
        return s["views"]
    if kind == "solve":
        if c["wait"]:
            return s["stats"].solve(LAM, delta_w=s["dw"])
        return s["stats"].solve_async(LAM, delta_w=s["dw"])
    if kind == "batch":
        return s["stats"].solve(LAM, delta_w=s["dw"])
    if kind == "project":
        return ispa.project(s["a"], s["w"], out_dtype=DTYPES[c["out"]])
    if kind == "w8a8":
        q_a, scale_a = ispa.quantize_rows(s["a"])
        return ispa.project_w8a8(q_a, scale_a, s["q_w"], s["scale_w"], out_dtype=DTYPES[c["out"]]), q_a, scale_a
    s["w"].copy_(s["w0"])  # a recalibration starts from the original weight
    ispa.inject_modulation(s["w"], s["dw"], transposed=True)
    kv = ispa.LocalKV(s["k"], s["v"], c["cache_len"], c["window"], c["sink"], ring=s["ring"])
    kv.append(s["k_new"], s["v_new"])
    out, lse = kv.attend(s["q"], c["heads"])
    y = ispa.project(out.to(BF16), s["w"], out_dtype=BF16)
    return {"y": y, "out": out, "lse": lse, "w": s["w"], "k": kv.k, "v": kv.v}


# -------------------------------------------------------- what a pass needs
def _key_sets(c):
    """(local keys, all keys) as lists of [begin, end)."""
    n, lo = c["cache_len"], max(0, c["cache_len"] - c["window"])
    sink = min(c["sink"], n)
    local = [(0, n)] if lo <= sink else [(b, e) for b, e in ((0, sink), (lo, n)) if e > b]
    return local, [(0, n)]


def work(case):
    c, kind = case, case["kind"]
    if kind == "attn":
        local, full = _key_sets(c)
        keys = sum(e - b for b, e in (full if c["dual"] else local))
        hidden, n_q = c["heads"] * c["head_dim"], c["n_q"]
        outs = 2 if c["dual"] else 1
        return {"bytes": 2 * hidden * (n_q + 2 * keys) + outs * 4 * n_q * (hidden + c["heads"]),
                "flops": 4 * n_q * keys * hidden}
    if kind in ("accum", "solve", "batch"):
        m, di, do = c["rows"], c["d_in"], c["d_out"]
        tri = di * (di + 1) // 2
        if kind == "accum":
            size = {"bf16": 2, "f32": 4}
            return {"bytes": m * (di * size[c["x"]] + 2 * do * size[c["y"]]) + 4 * (tri + di * do),
                    "flops": m * di * (di + 1) + 2 * m * di * do}
        layers = c.get("layers", 1)
        return {"bytes": layers * 4 * (tri + 2 * di * do), "flops": layers * (di**3 // 3 + 2 * di * di * do)}
    if kind in ("project", "w8a8"):
        m, di, do = c["rows"], c["d_in"], c["d_out"]
        out = m * do * (2 if c["out"] == "bf16" else 4)
        if kind == "project":
            return {"bytes": 2 * di * (m + do) + out, "flops": 2 * m * di * do}
        # the codes and scales are outputs of the pass as well
        return {"bytes": 2 * m * di + m * (di + 4) + do * (di + 4) + out, "flops": 2 * m * di * do}
    hidden, n_q = c["heads"] * c["head_dim"], c["n_q"]
    sink = min(c["sink"], c["cache_len"])
    kept = min(c["window"], c["cache_len"] - sink)
    keys = sink + min(kept + n_q, c["window"])
    stay = keys - min(n_q, c["window"])  # rows of the cache that are still held after the append
    return {"bytes": 2 * hidden * (2 * stay + 2 * min(n_q, c["window"]) + 2 * keys) + hidden * hidden * 8
            + 2 * hidden * n_q + 4 * n_q * (hidden + c["heads"]) + 2 * n_q * hidden,
            "flops": 4 * n_q * keys * hidden + 2 * n_q * hidden * hidden}


def tolerance(case):
    kind = case["kind"]
    # 16-bit softmax weights or results, fp32 sums: against 64 bits the rounding
    # shows as 1.7e-3 (attention, a bf16 result) and 3.3e-3 (both in turn)
    if kind in ("attn", "project"):
        return {"rel": 7e-3, "max": 8e-2}
    if kind == "convert":
        return {"rel": 1.3e-2, "max": 8e-2}
    if kind == "w8a8":  # integer product, fp32 scaling, one rounding: the codes are whole values
        return {"rel": 1e-5, "max": 1e-2}
    if kind == "accum":  # products of bf16 values in fp32 sums over the rows: 2e-7 against 64 bits
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 2e-5, "max": 1e-3}  # fp32 rounding times the conditioning of G: up to 2e-6 against 64 bits


# --------------------------------------------------------- the same in 64 bits
def _exact_attn(q, k, v, heads, sets):
    n_q, hidden = q.shape
    d = hidden // heads
    idx = torch.cat([torch.arange(b, e, device=q.device) for b, e in sets])
    out = torch.empty((n_q, hidden), dtype=F64, device=q.device)
    lse = torch.empty((heads, n_q), dtype=F64, device=q.device)
    for h in range(heads):
        col = slice(h * d, (h + 1) * d)
        kh, vh = k[idx, col].to(F64), v[idx, col].to(F64)
        for r in range(0, n_q, 1024):
            p = (q[r:r + 1024, col].to(F64) @ kh.t()) / math.sqrt(d)
            m = p.amax(dim=1, keepdim=True)
            p.sub_(m).exp_()
            z = p.sum(dim=1, keepdim=True)
            out[r:r + 1024, col] = (p @ vh) / z
            lse[h, r:r + 1024] = (m + z.log()).squeeze(1)
    return out, lse


def _exact_stats(x, y_full, y_local):
    xb = x.to(BF16).to(F64)
    r = (y_full.to(F32) - y_local.to(F32)).to(BF16).to(F64)  # R as the method stores it
    return xb.t() @ xb, xb.t() @ r, r.square().sum().reshape(1)


def _exact_solve(x, y_full, y_local):
    G, C, s = _exact_stats(x, y_full, y_local)
    lam = float(torch.tensor(LAM, dtype=F32))
    A = G + lam * torch.eye(G.shape[0], dtype=F64, device=G.device)
    dw = torch.cholesky_solve(C, torch.linalg.cholesky(A))
    return dw, s - (dw * C).sum() - lam * dw.square().sum()


def exact(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "attn":
        q, k, v = _qkv(c, g, c["cache_len"])
        local, full = _key_sets(c)
        if not c["dual"]:
            return _exact_attn(q, k, v, c["heads"], local)
        return _exact_attn(q, k, v, c["heads"], full) + _exact_attn(q, k, v, c["heads"], local)
    if kind == "accum":
        x, y_full, y_local = _warmup_rows(g, c["rows"], c["d_in"], c["d_out"])
        G, C, s = _exact_stats(x.to(DTYPES[c["x"]]), y_full.to(DTYPES[c["y"]]), y_local.to(DTYPES[c["y"]]))
        return {"G": _lower(G), "C": C, "s": s}
    if kind == "solve":
        dw, eps = _exact_solve(*_warmup_rows(g, c["rows"], c["d_in"], c["d_out"]))
        return (dw, float(eps)) if c["wait"] else (dw, eps, None)
    if kind == "batch":
        got = [_exact_solve(*_warmup_rows(g, c["rows"], c["d_in"], c["d_out"])) for _ in range(c["layers"])]
        return torch.stack([dw for dw, _ in got]), torch.cat([e for _, e in got]), None
    if kind in ("project", "w8a8"):
        a, w = _project_inputs(c, g)
        if kind == "project":
            return a.to(F64) @ w.to(F64).t()
        (q_a, s_a), (q_w, s_w) = _exact_codes(a), _exact_codes(w)
        return (q_a @ q_w.t()) * s_a.to(F64)[:, None] * s_w.to(F64)[None, :], None, s_a.to(F64)
    q, k, v, k_new, v_new, w0, dw = _convert_inputs(c, g)
    w = w0.to(F64) + dw.to(F64).t()
    n, window = c["cache_len"], c["window"]
    sink = min(c["sink"], n)
    recent = [torch.cat([old[max(sink, n - window):n], new])[-window:] for old, new in ((k, k_new), (v, v_new))]
    held = [torch.cat([old[:sink], tail]) for old, tail in zip((k, v), recent)]
    out, lse = _exact_attn(q, held[0], held[1], c["heads"], [(0, held[0].shape[0])])
    return {"y": out @ w.t(), "out": out, "lse": lse, "w": w, "k": None, "v": None}


def _exact_codes(x):
    """Per-row int8 codes as the scheme defines them (an fp32 quotient)."""
    x = x.to(F32)
    top = x.abs().amax(dim=1)
    scale = torch.where(top > 0, top / 127.0, torch.ones_like(top))
    return torch.round(x / scale[:, None]).clamp_(-127, 127).to(F64), scale
