"""The work that a user of the engine has it do, as cases to time and to compare.

Four kinds, each through public entry points of the package:

  step   one engine call on a decoder: a decode step of a batch, or a mixed step in which some sequences take an
         observation chunk while the others decode (continuous batching).  Every request continues a shared prompt:
         it is forked from a resident sequence, stepped and freed, so that a pass leaves the cache as it found it.
         The fused layers of a decode batch and of a long pass are reached through these calls only.
  ffn    the feed-forward half of a layer at kernel level: RMSNorm + gate/up + SwiGLU, then down + residual.
  attn   paged decode attention of one layer, one query per sequence.
  chunk  the attention half of a layer for prefill segments: q-k-v projection, rotary embedding and cache append,
         chunk attention, output projection + residual.

Shapes are the repository's own decoder shapes; contexts, batch sizes and chunk lengths are those of its workloads
(batch 1 at a context of some 1500 tokens, 32 sequences U[512, 8192], observations of 128 .. 512 tokens in chunks of
256, a 2048-token chunk beside 63 decode rows, the attention micro-benchmark at batch 16, U[256, 4096]).  Block
tables are seeded permutations of the pool.  Passes of 512 rows or more give the layer matrices' fp16 copy, as the
benchmark does; shorter ones keep two bf16 terms.
"""
import math

import numpy as np
import torch

import paper_2406_00059_amd as ld
from workloads import LLAMA7B, LLAMA13B, MISTRAL7B, TINY

SHAPES = {"tiny": TINY, "7b": LLAMA7B, "7b-gqa": MISTRAL7B, "13b": LLAMA13B}
F16_ROWS = 512      # rows from which a pass may take its rows as one fp16 term


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: a two-layer fp32 decoder, one token; launches and latency are all there is
        {"name": "step_tiny_1", "kind": "step", "shape": "tiny", "layers": 2, "dec": 1, "pf": 0, "pf_rows": 0,
         "ctx_lo": 32, "ctx_hi": 32},
        # the headline workload: one token of the whole 7B decoder at batch 1, in the middle of a tool-call session
        {"name": "step_7b_1", "kind": "step", "shape": "7b", "layers": 32, "dec": 1, "pf": 0, "pf_rows": 0,
         "ctx_lo": 1520, "ctx_hi": 1520},
        # a decode step of the continuous-batching workload (four of its layers, whole batch and contexts)
        {"name": "step_7b_32", "kind": "step", "shape": "7b", "layers": 4, "dec": 32, "pf": 0, "pf_rows": 0,
         "ctx_lo": 512, "ctx_hi": 8192},
        # its mixed step: 28 decode rows beside four observations of 256 tokens behind their pending token
        {"name": "step_7b_mixed", "kind": "step", "shape": "7b", "layers": 4, "dec": 28, "pf": 4, "pf_rows": 257,
         "ctx_lo": 512, "ctx_hi": 8192},
        # feed-forward of one decoded token
        {"name": "ffn_7b_1", "kind": "ffn", "shape": "7b", "rows": 1},
        # feed-forward of a small decode batch, not a multiple of any tile
        {"name": "ffn_7b_20", "kind": "ffn", "shape": "7b", "rows": 20},
        # feed-forward of a short observation, appended in one pass
        {"name": "ffn_7b_152", "kind": "ffn", "shape": "7b", "rows": 152},
        # feed-forward of the largest pass: 63 decode rows beside a 2048-token chunk on the 13B shape
        {"name": "ffn_13b_2111", "kind": "ffn", "shape": "13b", "rows": 2111},
        # the decode-attention micro-benchmark
        {"name": "attn_7b_16", "kind": "attn", "shape": "7b", "rows": 16, "ctx_lo": 256, "ctx_hi": 4096},
        # decode attention of the batch-32 workload on grouped KV heads with an attention band
        {"name": "attn_gqa_32", "kind": "attn", "shape": "7b-gqa", "rows": 32, "ctx_lo": 512, "ctx_hi": 8192},
        # attention half of a layer for one 256-row chunk of an observation in the batch-1 session
        {"name": "chunk_7b_256", "kind": "chunk", "shape": "7b", "segs": 1, "seg_rows": 256, "ctx_lo": 1500, "ctx_hi": 1500},
        # the same for the four observations of a mixed step behind long contexts
        {"name": "chunk_7b_1028", "kind": "chunk", "shape": "7b", "segs": 4, "seg_rows": 257, "ctx_lo": 512, "ctx_hi": 8192},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges: batch sizes and row counts over their logarithm, ragged lengths."""
    kind = rng.choice(["step", "ffn", "ffn", "attn", "chunk"])
    if kind == "ffn":
        shape = rng.choice(["7b", "7b-gqa", "13b"])
        return {"kind": kind, "shape": shape, "rows": _log_int(rng, 1, 2110)}
    lo = _log_int(rng, 16, 4096)
    if kind == "attn":
        return {"kind": kind, "shape": rng.choice(["7b", "7b-gqa", "13b"]), "rows": _log_int(rng, 1, 40), "ctx_lo": lo,
                "ctx_hi": rng.randint(lo, 8192)}
    if kind == "chunk":
        return {"kind": kind, "shape": rng.choice(["7b", "7b-gqa"]), "segs": rng.randint(1, 4),
                "seg_rows": _log_int(rng, 48, 300), "ctx_lo": lo, "ctx_hi": rng.randint(lo, 8192)}
    pf = rng.choice([0, 0, 1, 2, 4])
    return {"kind": kind, "shape": rng.choice(["7b", "7b", "7b-gqa", "tiny"]), "layers": 2, "dec": _log_int(rng, 1, 28),
            "pf": pf, "pf_rows": rng.randint(40, 257) if pf else 0, "ctx_lo": lo, "ctx_hi": rng.randint(lo, 8192)}


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)


def _normal(g, shape, dtype=torch.float32, std=1.0, mean=0.0):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)


def _el(sh):
    return torch.float32 if sh.dtype == "f32" else torch.bfloat16


def _weights(sh, g):
    """N(0, 0.02^2) matrices, gains 1 + 0.02 N(0,1) in float32 (the repository's recipe)."""
    d, f, e = sh.d_model, sh.d_ffn, _el(sh)
    nq, nkv = sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim
    w = {"embed": _normal(g, (sh.vocab, d), e, 0.02), "lm_head": _normal(g, (sh.vocab, d), e, 0.02),
         "final_norm": _normal(g, (d,), std=0.02, mean=1.0)}
    for k, s in (("wqkv", (nq + 2 * nkv, d)), ("wo", (d, nq)), ("wgate_up", (2 * f, d)), ("wdown", (d, f))):
        w[k] = [_normal(g, s, e, 0.02) for _ in range(sh.n_layers)]
    for k in ("attn_norm", "ffn_norm"):
        w[k] = [_normal(g, (d,), std=0.02, mean=1.0) for _ in range(sh.n_layers)]
    return w


def _lengths(n, lo, hi):
    """Context lengths of a case, uniform in [lo, hi]: a function of the case, so that buffers have the same shapes for
    every seed."""
    return [int(v) for v in np.random.RandomState((n * 8209 + lo) * 8209 + hi).randint(lo, hi + 1, n)]


def _step_contexts(case):
    return [max(16, c // 16 * 16) for c in _lengths(case["dec"] + case["pf"], case["ctx_lo"], case["ctx_hi"])]      # whole blocks are shared


def _step_inputs(case, seed):
    sh = SHAPES[case["shape"]].with_layers(case["layers"])
    rs, g = np.random.RandomState(seed % (1 << 31)), _gen(seed)
    n = case["dec"] + case["pf"]
    ctx = _step_contexts(case)
    new = [1] * case["dec"] + [case["pf_rows"]] * case["pf"]      # rows a sequence feeds
    n_blocks = sum(c // 16 for c in ctx) + sum(r // 16 + 1 for r in new)
    perm = rs.permutation(n_blocks)
    tables, at = [], 0
    for c in ctx:
        tables.append(perm[at:at + c // 16].astype(np.int32))
        at += c // 16
    tokens = [rs.randint(0, sh.vocab, r).astype(np.int32) for r in new]
    w = _weights(sh, g)
    pool = _normal(g, (sh.n_layers, n_blocks, 2, sh.n_kv_heads, 16, sh.head_dim), _el(sh))
    return sh, w, pool, n_blocks, ctx, new, tables, tokens


def _step_prepare(case, seed):
    sh, w, pool, n_blocks, ctx, new, tables, tokens = _step_inputs(case, seed)
    n, rows = len(ctx), sum(new)
    model = ld.Model(sh, w)
    blocks = max(-(-(c + r) // 16) for c, r in zip(ctx, new))
    kv = ld.KV(model, n_blocks, rows, 2 * n, blocks, pool=pool)
    if rows >= F16_ROWS:
        model.attach_f16_image()
    parents = []
    for c, t in zip(ctx, tables):
        s = ld.ld_kv_alloc(kv.h)
        for j, b in enumerate(t):
            ld.ld_kv_map(kv.h, s, j, int(b))
        ld.ld_kv_assume(kv.h, s, c)
        parents.append(s)
    return {"kind": "step", "model": model, "kv": kv, "parents": parents, "ctx": ctx, "tokens": tokens, "dec": case["dec"],
            "vocab": sh.vocab}


def _step_run(s):
    kv, nd = s["kv"].h, s["dec"]
    seqs = []
    for p, c, t in zip(s["parents"], s["ctx"], s["tokens"]):
        q = ld.ld_kv_fork(kv, p, c)
        ld.ld_kv_assume(kv, q, 0, int(t[0]))      # the token it emitted last
        seqs.append(q)
    take = lambda seq, token, pos: 0      # where a parser reads the tokens
    if len(seqs) == nd:
        _, logits = ld.ld_decode_step(kv, seqs, callback=take, logits_vocab=s["vocab"])
    else:
        _, logits = ld.ld_step_mixed(kv, seqs[:nd], seqs[nd:], [t[1:] for t in s["tokens"][nd:]], callback=take,
                                     logits_vocab=s["vocab"])
    for q in reversed(seqs):
        ld.ld_kv_free(kv, q)
    return logits


def _ffn_inputs(case, seed):
    sh, g, rows = SHAPES[case["shape"]], _gen(seed), case["rows"]
    return sh, {"gain": _normal(g, (sh.d_model,), std=0.02, mean=1.0),
                "wgu": _normal(g, (2 * sh.d_ffn, sh.d_model), torch.bfloat16, 0.02),
                "wd": _normal(g, (sh.d_model, sh.d_ffn), torch.bfloat16, 0.02), "x": _normal(g, (rows, sh.d_model))}


def _image(w, flag):
    h = torch.empty_like(w, dtype=torch.float16)
    ld.ldk_weights_to_f16(w, h, flag)
    return h


def _scratch(*sizes):
    n = max(sizes)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _ffn_prepare(case, seed):
    sh, s = _ffn_inputs(case, seed)
    rows = case["rows"]
    s.update(kind="ffn", eps=sh.rms_eps, act=torch.empty(rows, sh.d_ffn, device="cuda"), y=torch.empty_like(s["x"]),
             scratch=_scratch(ld.ldk_linear_scratch_bytes(rows, sh.d_ffn, sh.d_model, ld.LDK_SWIGLU),
                              ld.ldk_linear_scratch_bytes(rows, sh.d_model, sh.d_ffn, ld.LDK_ADD)))
    if rows >= F16_ROWS:
        s["flag"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        s["wgu16"], s["wd16"] = _image(s["wgu"], s["flag"]), _image(s["wd"], s["flag"])
    return s


def _ffn_run(s):
    s["y"].copy_(s["x"])      # the residual stream
    if "flag" in s:
        ld.ldk_linear_f16(s["wgu"], s["x"], s["act"], s["flag"], ld.LDK_SWIGLU, s["gain"], s["eps"], s["scratch"], W_f16=s["wgu16"])
        ld.ldk_linear_f16(s["wd"], s["act"], s["y"], s["flag"], ld.LDK_ADD, scratch=s["scratch"], W_f16=s["wd16"])
        return {"act": s["act"], "y": s["y"], "overflow": s["flag"]}
    ld.ldk_linear(s["wgu"], s["x"], s["act"], ld.LDK_SWIGLU, s["gain"], s["eps"], s["scratch"])
    ld.ldk_linear(s["wd"], s["act"], s["y"], ld.LDK_ADD, scratch=s["scratch"])
    return {"act": s["act"], "y": s["y"]}


def _paged(sh, rs, g, lengths):
    """One layer's pool and block table for sequences of these lengths: a seeded permutation of the blocks."""
    nb = [-(-n // 16) for n in lengths]
    perm = rs.permutation(sum(nb))
    table = np.zeros((len(nb), max(nb)), dtype=np.int32)
    at = 0
    for i, n in enumerate(nb):
        table[i, :n] = perm[at:at + n]
        at += n
    pool = _normal(g, (sum(nb), 2, sh.n_kv_heads, 16, sh.head_dim), torch.bfloat16)
    return pool, torch.from_numpy(table).cuda()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _attn_inputs(case, seed):
    sh, g, rs = SHAPES[case["shape"]], _gen(seed), np.random.RandomState(seed % (1 << 31))
    ctx = _lengths(case["rows"], case["ctx_lo"], case["ctx_hi"])
    pool, table = _paged(sh, rs, g, ctx)
    return sh, ctx, {"pool": pool, "table": table, "q": _normal(g, (case["rows"], sh.n_heads * sh.head_dim))}


def _attn_prepare(case, seed):
    sh, ctx, s = _attn_inputs(case, seed)
    r = case["rows"]
    s.update(kind="attn", sh=sh, max_ctx=max(ctx), ctx=_dev(ctx), slot=_dev(np.arange(r)), out=torch.empty_like(s["q"]),
             scratch=_scratch(ld.ldk_attention_scratch_bytes(r, sh.n_heads, sh.n_kv_heads, sh.head_dim, max(ctx), sh.window)))
    return s


def _attn_run(s):
    sh = s["sh"]
    ld.ldk_paged_attention(s["q"], sh.n_heads * sh.head_dim, s["pool"], s["table"], s["slot"], s["ctx"], s["max_ctx"], sh.n_heads,
                           sh.n_kv_heads, sh.head_dim, s["out"], s["scratch"], window=sh.window)
    return s["out"]


def _chunk_inputs(case, seed):
    sh, g, rs = SHAPES[case["shape"]], _gen(seed), np.random.RandomState(seed % (1 << 31))
    ctx, n = _lengths(case["segs"], case["ctx_lo"], case["ctx_hi"]), case["seg_rows"]
    pool, table = _paged(sh, rs, g, [c + n for c in ctx])
    nq, nkv = sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim
    return sh, ctx, {"pool": pool, "table": table, "x": _normal(g, (n * len(ctx), sh.d_model)),
                     "gain": _normal(g, (sh.d_model,), std=0.02, mean=1.0),
                     "wqkv": _normal(g, (nq + 2 * nkv, sh.d_model), torch.bfloat16, 0.02),
                     "wo": _normal(g, (sh.d_model, nq), torch.bfloat16, 0.02)}


def _chunk_prepare(case, seed):
    sh, ctx, s = _chunk_inputs(case, seed)
    n = case["seg_rows"]
    rows, nqkv, nq = n * len(ctx), s["wqkv"].shape[0], sh.n_heads * sh.head_dim
    tiles = [(i * n + r, min(128, n - r), c + r, i) for i, c in enumerate(ctx) for r in range(0, n, 128)]
    pos = np.concatenate([np.arange(c, c + n) for c in ctx])
    s.update(kind="chunk", sh=sh, tiles=_dev(tiles), pos=_dev(pos), slot=_dev(np.repeat(np.arange(len(ctx)), n)),
             max_pos=int(pos.max()), cs=torch.empty(rows, sh.head_dim, device="cuda"), qkv=torch.empty(rows, nqkv, device="cuda"),
             att=torch.empty(rows, nq, device="cuda"), y=torch.empty_like(s["x"]),
             scratch=_scratch(ld.ldk_linear_scratch_bytes(rows, nqkv, sh.d_model, ld.LDK_STORE),
                              ld.ldk_linear_scratch_bytes(rows, sh.d_model, nq, ld.LDK_ADD)),
             att_scratch=_scratch(ld.ldk_prefill_attention_scratch_bytes()))
    ld.ldk_rope_table(s["pos"], sh.head_dim, sh.rope_base, s["cs"])      # once for all layers of a pass
    if rows >= F16_ROWS:
        s["flag"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        s["wqkv16"], s["wo16"] = _image(s["wqkv"], s["flag"]), _image(s["wo"], s["flag"])
    return s


def _chunk_run(s):
    sh = s["sh"]
    H, Hkv, hd = sh.n_heads, sh.n_kv_heads, sh.head_dim
    nqkv = s["qkv"].shape[1]
    s["y"].copy_(s["x"])      # the residual stream
    if "flag" in s:
        ld.ldk_linear_f16(s["wqkv"], s["x"], s["qkv"], s["flag"], ld.LDK_STORE, s["gain"], sh.rms_eps, s["scratch"], W_f16=s["wqkv16"])
        ld.ldk_rope_kv_write(s["qkv"], s["cs"], s["pos"], s["slot"], s["table"], s["pool"], H, Hkv, hd)
        ld.ldk_prefill_attention_f16(s["qkv"], nqkv, s["pool"], s["table"], s["tiles"], H, Hkv, hd, s["att"], s["max_pos"], s["flag"],
                                     window=sh.window, scratch=s["att_scratch"])
        ld.ldk_linear_f16(s["wo"], s["att"], s["y"], s["flag"], ld.LDK_ADD, scratch=s["scratch"], W_f16=s["wo16"])
        return {"att": s["att"], "y": s["y"], "pool": s["pool"], "overflow": s["flag"]}
    ld.ldk_qkv_rope(s["wqkv"], s["x"], s["qkv"], s["cs"], s["pos"], s["slot"], s["table"], s["pool"], H, Hkv, hd, s["gain"],
                    sh.rms_eps, s["scratch"])
    ld.ldk_prefill_attention(s["qkv"], nqkv, s["pool"], s["table"], s["tiles"], H, Hkv, hd, s["att"], s["max_pos"],
                             window=sh.window, scratch=s["att_scratch"])
    ld.ldk_linear(s["wo"], s["att"], s["y"], ld.LDK_ADD, scratch=s["scratch"])
    return {"att": s["att"], "y": s["y"], "pool": s["pool"]}


def prepare(case, seed):
    return {"step": _step_prepare, "ffn": _ffn_prepare, "attn": _attn_prepare, "chunk": _chunk_prepare}[case["kind"]](case, seed)


def run(state):
    return {"step": _step_run, "ffn": _ffn_run, "attn": _attn_run, "chunk": _chunk_run}[state["kind"]](state)


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    sh = SHAPES[case["shape"]]
    e = 4 if sh.dtype == "f32" else 2
    d, f, nq, nkv = sh.d_model, sh.d_ffn, sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim
    seen = lambda c: min(c, sh.window) if sh.window else c
    if case["kind"] == "ffn":
        t = case["rows"]
        return {"bytes": 3 * d * f * e + 4 * t * (2 * d + f), "flops": 6 * t * d * f}
    if case["kind"] == "attn":
        ctx = [seen(c) for c in _lengths(case["rows"], case["ctx_lo"], case["ctx_hi"])]
        return {"bytes": sum(ctx) * 2 * nkv * e + 8 * len(ctx) * nq, "flops": 4 * sum(ctx) * nq}
    # rows that attend, cached positions that are read and (row, position) pairs that are multiplied
    if case["kind"] == "chunk":
        feeds = [(c, case["seg_rows"]) for c in _lengths(case["segs"], case["ctx_lo"], case["ctx_hi"])]
    else:
        feeds = list(zip(_step_contexts(case), [1] * case["dec"] + [case["pf_rows"]] * case["pf"]))
    t = sum(r for _, r in feeds)
    read = sum(min(c, sh.window - 1) if sh.window else c for c, _ in feeds)
    pairs = sum(seen(p + 1) for c, r in feeds for p in range(c, c + r))
    proj = (2 * nq + 2 * nkv) * d
    if case["kind"] == "chunk":
        return {"bytes": proj * e + (read + t) * 2 * nkv * e + t * (8 * d + 4 * nq), "flops": 2 * t * proj + 4 * pairs * nq}
    n, layers = len(feeds), case["layers"]
    return {"bytes": layers * e * (proj + 3 * d * f + (read + t) * 2 * nkv) + e * sh.vocab * d + 4 * n * sh.vocab,
            "flops": layers * (2 * t * (proj + 3 * d * f) + 4 * pairs * nq) + 2 * n * sh.vocab * d}


def tolerance(case):
    """About four times the distance to 64 bits that was measured.  Two bf16 terms carry 16 bits of an activation, one
    fp16 term (passes of 512 rows or more) 11; where keys and values are appended, those that lie next to a rounding
    boundary of the cache's type go to either side of it."""
    if case["kind"] == "step":
        if case["shape"] == "tiny":
            return {"rel": 2e-6}
        long = case["dec"] + case["pf"] * case["pf_rows"] >= F16_ROWS
        return {"rel": 5e-3 if long else 2e-4}
    if case["kind"] == "ffn":
        return {"rel": 1.4e-3 if case["rows"] >= F16_ROWS else 1.6e-5 if case["rows"] > 1 else 1e-6}
    if case["kind"] == "attn":
        sh = SHAPES[case["shape"]]
        return {"rel": 1e-6 if sh.n_heads == sh.n_kv_heads else 1.3e-5}
    return {"rel": 4e-3 if case["segs"] * case["seg_rows"] >= F16_ROWS else 6e-4}


# ---------------------------------------------------------------- the same in 64 bits

def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + float(np.float32(eps))) * g.double()


def _mm(x, w):
    """x w^T in float64, the matrix widened a part at a time."""
    return torch.cat([x @ p.double().t() for p in w.split(8192)], 1)


def _rotate(x, pos, sh):
    """x [T, heads, hd]: pairs (i, i + hd / 2) by the position's angles."""
    half = sh.head_dim // 2
    theta = sh.rope_base ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / sh.head_dim)
    a = pos.double()[:, None, None] * theta
    u, v = x[..., :half], x[..., half:]
    return torch.cat([u * a.cos() - v * a.sin(), u * a.sin() + v * a.cos()], -1)


def _history(pool, blocks, n):
    """Keys and values [Hkv, n, hd] of a sequence's first n positions, from one layer's pool (values lie transposed)."""
    p = pool[blocks.long()].double()
    nb, _, hkv, _, hd = p.shape
    k = p[:, 0].permute(1, 0, 2, 3).reshape(hkv, nb * 16, hd)
    v = p[:, 1].reshape(nb, hkv, hd, 16).permute(1, 0, 3, 2).reshape(hkv, nb * 16, hd)
    return k[:, :n], v[:, :n]


def _attend(q, k, v, pos, window):
    """q [R, H, hd] at positions pos over k, v [Hkv, n, hd]."""
    h, hkv = q.shape[1], k.shape[0]
    out = torch.empty_like(q)
    j = torch.arange(k.shape[1], device="cuda")
    ok = j[None] <= pos[:, None]
    if window:
        ok &= j[None] > pos[:, None] - window
    for i in range(hkv):
        own = slice(i * (h // hkv), (i + 1) * (h // hkv))
        s = (q[:, own] @ k[i].t()) / math.sqrt(q.shape[-1])
        out[:, own] = torch.softmax(s.masked_fill(~ok[:, None], -math.inf), -1) @ v[i]
    return out


def _split_qkv(qkv, pos, sh):
    """Rotated queries, and the keys and values as the cache keeps them."""
    h, hkv, hd = sh.n_heads, sh.n_kv_heads, sh.head_dim
    x = qkv.reshape(len(qkv), h + 2 * hkv, hd)
    keep = lambda t: t.to(_el(sh)).double()
    return _rotate(x[:, :h], pos, sh), keep(_rotate(x[:, h:h + hkv], pos, sh)), keep(x[:, h + hkv:])


def exact(case, seed):
    return {"step": _step_exact, "ffn": _ffn_exact, "attn": _attn_exact, "chunk": _chunk_exact}[case["kind"]](case, seed)


def _ffn_exact(case, seed):
    sh, s = _ffn_inputs(case, seed)
    x = s["x"].double()
    gu = _mm(_rms(x, s["gain"], sh.rms_eps), s["wgu"])
    act = torch.nn.functional.silu(gu[:, :sh.d_ffn]) * gu[:, sh.d_ffn:]
    out = {"act": act, "y": x + _mm(act, s["wd"])}
    if case["rows"] >= F16_ROWS:
        out["overflow"] = None
    return out


def _attn_exact(case, seed):
    sh, ctx, s = _attn_inputs(case, seed)
    q = s["q"].double().reshape(-1, sh.n_heads, sh.head_dim)
    out = []
    for i, c in enumerate(ctx):
        k, v = _history(s["pool"], s["table"][i, :-(-c // 16)], c)
        out.append(_attend(q[i:i + 1], k, v, torch.tensor([c - 1], device="cuda"), sh.window).reshape(1, -1))
    return torch.cat(out)


def _chunk_exact(case, seed):
    sh, ctx, s = _chunk_inputs(case, seed)
    n = case["seg_rows"]
    x = s["x"].double()
    qkv = _mm(_rms(x, s["gain"], sh.rms_eps), s["wqkv"])
    att, pool = [], s["pool"].clone()
    for i, c in enumerate(ctx):
        pos = torch.arange(c, c + n, device="cuda")
        q, k_new, v_new = _split_qkv(qkv[i * n:(i + 1) * n], pos, sh)
        blocks = s["table"][i, :-(-(c + n) // 16)]
        phys = blocks[pos // 16].long()
        pool[phys, 0, :, pos % 16] = k_new.to(pool.dtype)
        pool.view(pool.shape[0], 2, sh.n_kv_heads, sh.head_dim, 16)[phys, 1, :, :, pos % 16] = v_new.to(pool.dtype)
        k, v = _history(pool, blocks, c + n)
        att.append(_attend(q, k, v, pos, sh.window).reshape(n, -1))
    att = torch.cat(att)
    out = {"att": att, "y": x + _mm(att, s["wo"]), "pool": pool}
    if n * len(ctx) >= F16_ROWS:
        out["overflow"] = None
    return out


def _step_exact(case, seed):
    sh, w, pool, _, ctx, new, tables, tokens = _step_inputs(case, seed)
    pos = torch.cat([torch.arange(c, c + r, device="cuda") for c, r in zip(ctx, new)])
    x = w["embed"][torch.from_numpy(np.concatenate(tokens)).cuda().long()].double()
    for l in range(sh.n_layers):
        q, k_new, v_new = _split_qkv(_mm(_rms(x, w["attn_norm"][l], sh.rms_eps), w["wqkv"][l]), pos, sh)
        att, at = [], 0
        for c, r, t in zip(ctx, new, tables):
            k, v = _history(pool[l], torch.from_numpy(t).cuda(), c)
            own = slice(at, at + r)
            at += r
            k, v = torch.cat([k, k_new[own].transpose(0, 1)], 1), torch.cat([v, v_new[own].transpose(0, 1)], 1)
            att.append(_attend(q[own], k, v, pos[own], sh.window).reshape(r, -1))
        x = x + _mm(torch.cat(att), w["wo"][l])
        gu = _mm(_rms(x, w["ffn_norm"][l], sh.rms_eps), w["wgate_up"][l])
        x = x + _mm(torch.nn.functional.silu(gu[:, :sh.d_ffn]) * gu[:, sh.d_ffn:], w["wdown"][l])
    last = torch.from_numpy(np.cumsum(new) - 1).cuda()
    return _mm(_rms(x[last], w["final_norm"], sh.rms_eps), w["lm_head"])
