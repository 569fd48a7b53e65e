"""Workloads by which the speed of the library is measured.

Every case is one call (or one request of a few layers) through the public
Python entry points, at sizes from the seeded workloads, the tests and the
benchmark of this repository, with ragged ones between them.  The kinds:

layer   one Re-Prefill layer step on an HBM-resident prefix (score, select,
        attend in place) through ``Context.reprefill_layer``; bf16, or fp32
host    one request of a few layers on a prefix in pinned host memory: the
        next layer's chunks prefetched, the mispredicted ones fetched on demand
score   chunk scoring alone (``score_chunks``)
select  top-k selection alone (``select_topk_chunks``)
gather  the kept chunks' spans into compact buffers (``gather_chunks``)
attn    attention over compact kept chunks (``sparse_prefill_attn``)

Inputs stand for post-RoPE Q, K and V: unit normal noise, a shared direction
per KV head in every query, and the same direction added to the keys of 5% of
the chunks (the ones that draw attention), which drift from layer to layer.
"""
from __future__ import annotations

import math

import torch

import paper_2601_13631_amd as ckv

DEV = "cuda"

# (query heads, KV heads, head_dim) of the bf16 shapes: Qwen2.5-0.5B, 7B and
# 14B/32B attention layers, then two generic ones
HEADS = ((14, 2, 64), (28, 4, 128), (40, 8, 128), (32, 8, 128), (12, 4, 64))


def _case(name, kind, n, s, heads, c, keep, dtype="bf16", layers=1):
    return {"name": name, "kind": kind, "n": n, "s": s, "hq": heads[0], "hkv": heads[1],
            "d": heads[2], "c": c, "keep": keep, "dtype": dtype, "layers": layers}


def listed():
    return [
        # a short few-shot prompt with a short question: launches and latency count
        _case("layer_1k", "layer", 1000, 24, (14, 2, 64), 16, 0.25),
        # the fp32 configuration
        _case("layer_1k_f32", "layer", 1024, 32, (4, 1, 64), 16, 0.25, "f32"),
        # 0.5B-shaped layer, 8K prefix
        _case("layer_8k", "layer", 8192, 128, (14, 2, 64), 16, 0.20),
        # 7B-shaped layer, 32K prefix: the benchmark's default workload
        _case("layer_32k", "layer", 32768, 256, (28, 4, 128), 32, 0.10),
        # a one-line question on a long shared prefix, ragged sizes
        _case("layer_30k_short", "layer", 30011, 19, (28, 4, 128), 32, 0.10),
        # 14B-shaped layer, 64K prefix, fine chunks
        _case("layer_64k", "layer", 65536, 512, (40, 8, 128), 16, 0.15),
        # 32B-shaped layer, 128K prefix, long suffix: the largest
        _case("layer_128k", "layer", 131072, 1024, (40, 8, 128), 32, 0.10),
        # four 7B-shaped layers whose 32K prefix lives in pinned host memory
        _case("host_32k", "host", 32768, 256, (28, 4, 128), 32, 0.10, layers=4),
        # scoring alone at the finest chunks, ragged prefix
        _case("score_12k_c4", "score", 12345, 200, (14, 2, 64), 4, 0.10),
        # selection among the chunks of a 128K prefix at 8 tokens per chunk
        _case("select_16k", "select", 131072, 1, (40, 8, 128), 8, 0.10),
        # the kept spans of a 64K prefix made compact
        _case("gather_64k", "gather", 65536, 1, (40, 8, 128), 32, 0.15),
        # attention over many kept chunks of a ragged 16K prefix
        _case("attn_16k_half", "attn", 16000, 512, (32, 8, 128), 64, 0.50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "layer", "f32", "host", "score", "score",
                       "select", "gather", "attn", "attn"))
    heads = rng.choice(HEADS)
    c = rng.choice((8, 16, 32, 64))
    keep = round(rng.uniform(0.05, 0.30), 3)
    n, s = _log_int(rng, 1000, 131072), _log_int(rng, 8, 1024)
    if kind == "f32":  # the fp32 path: small prompts, four query heads
        return {"kind": "layer", "n": _log_int(rng, 300, 4096), "s": _log_int(rng, 4, 128), "hq": 4,
                "hkv": rng.choice((1, 2)), "d": 64, "c": rng.choice((8, 16, 32)),
                "keep": keep, "dtype": "f32", "layers": 1}
    if kind == "host":
        n, s, c = _log_int(rng, 4000, 32768), _log_int(rng, 16, 256), rng.choice((16, 32, 64))
    elif kind == "score":
        n, c = _log_int(rng, 1000, 65536), rng.choice((4, 8, 16, 32, 64, 96))
    elif kind == "select":
        c = rng.choice((4, 8, 16))
    elif kind == "attn":
        n, keep = _log_int(rng, 1000, 65536), round(rng.uniform(0.05, 0.60), 3)
    return {"kind": kind, "n": n, "s": 1 if kind in ("select", "gather") else s, "hq": heads[0],
            "hkv": heads[1], "d": heads[2], "c": c, "keep": keep, "dtype": "bf16",
            "layers": rng.randint(2, 4) if kind == "host" else 1}


# ---- inputs ------------------------------------------------------------------

def _generator(seed, salt):
    return torch.Generator(DEV).manual_seed(int(seed) * 1009 + salt)


def _sizes(case):
    m = ckv.num_chunks(case["n"], case["c"])
    return m, ckv.num_keep(m, case["keep"])


def _dims(case):
    return ckv.make_dims(case["n"], case["s"], case["hq"], case["hkv"], case["d"], case["c"],
                         ckv.DTYPE_F32 if case["dtype"] == "f32" else ckv.DTYPE_BF16)


def _heavy_chunks(case, seed, layer):
    """5% of the chunks; 15% of them change from one layer to the next."""
    m, _ = _sizes(case)
    h = max(1, round(0.05 * m))
    order = torch.randperm(m, generator=_generator(seed, 1), device=DEV)
    at = (torch.arange(h, device=DEV) + layer * math.ceil(0.15 * h)) % m
    return order[at]


def _tensors(case, seed, layer=0, names=("q", "k", "v", "ks", "vs")):
    """Q [S][Hq][d], prefix K/V [n][Hkv][d], suffix K/V [S][Hkv][d]."""
    n, s, hq, hkv, d, c = (case[x] for x in ("n", "s", "hq", "hkv", "d", "c"))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    g = _generator(seed, 100 + layer)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)

    u = torch.nn.functional.normalize(normal(hkv, d), dim=1)
    t = {}
    if "q" in names:
        t["q"] = (normal(s, hq, d) + u.repeat_interleave(hq // hkv, 0)).to(dt)
    if "k" in names:
        k = normal(n, hkv, d)
        heavy = torch.zeros(ckv.num_chunks(n, c), dtype=torch.bool, device=DEV)
        heavy[_heavy_chunks(case, seed, layer)] = True
        k += 1.5 * u * heavy.repeat_interleave(c)[:n, None, None]
        t["k"] = k.to(dt)
    if "v" in names:
        t["v"] = normal(n, hkv, d).to(dt)
    if "ks" in names:
        t["ks"], t["vs"] = normal(s, hkv, d).to(dt), normal(s, hkv, d).to(dt)
    return t


def _scores_like(case, seed):
    """Chunk scores as scoring gives them: a common level, 5% heavier chunks."""
    m, _ = _sizes(case)
    g = _generator(seed, 7)
    a = torch.exp(0.05 * torch.randn(m, generator=g, device=DEV, dtype=torch.float64))
    a[_heavy_chunks(case, seed, 0)] *= 1.6
    return a * (case["hq"] * 512.0 / m)


def _random_set(case, seed):
    m, k = _sizes(case)
    p = torch.randperm(m, generator=_generator(seed, 3), device=DEV)[:k]
    return torch.sort(p).values.to(torch.int32)


def _chunk_major(case, k, v):
    """Host store of one layer: chunk j is one span [K rows; V rows], padded with zeros."""
    m, _ = _sizes(case)
    n, hkv, d = k.shape
    c = case["c"]
    out = torch.zeros((m, 2, c, hkv, d), dtype=k.dtype, pin_memory=True)
    pad = torch.zeros((m * c - n, hkv, d), dtype=k.dtype, device=DEV)
    for i, x in enumerate((k, v)):
        out[:, i] = torch.cat((x, pad)).view(m, c, hkv, d).cpu()
    return out


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind, dims = case["kind"], _dims(case)
    m, k = _sizes(case)
    s, hkv, d, c = case["s"], case["hkv"], case["d"], case["c"]
    st = {"kind": kind, "dims": dims, "m": m, "n_kept": k}
    if kind in ("layer", "host"):
        st["layers"] = []
        for layer in range(case["layers"]):
            t = _tensors(case, seed, layer)
            if kind == "host":
                t["store"] = _chunk_major(case, t["k"], t.pop("v"))
            t["scores"] = torch.empty(m, dtype=torch.float64, device=DEV)
            t["sel"] = torch.empty(k, dtype=torch.int32, device=DEV)
            t["out"] = torch.empty_like(t["q"])
            st["layers"].append(t)
        st["ctx"] = ckv.Context(dims, case["layers"], case["keep"],
                                ckv.CTX_HOST_PREFIX if kind == "host" else 0)
        if kind == "host":
            st["ctx"].set_host_layers([t["store"] for t in st["layers"]])
    elif kind == "score":
        st.update(_tensors(case, seed, names=("q", "k")))
        st["scores"] = torch.empty(m, dtype=torch.float64, device=DEV)
        st["ws"] = _bytes(ckv.score_workspace_bytes(dims))
    elif kind == "select":
        st["scores"] = _scores_like(case, seed)
        st["sel"] = torch.empty(k, dtype=torch.int32, device=DEV)
        st["ws"] = _bytes(ckv.select_workspace_bytes(m))
    elif kind == "gather":
        st.update(_tensors(case, seed, names=("k", "v")))
        st["sel"] = _random_set(case, seed)
        st["k_sel"] = torch.empty((k * c, hkv, d), dtype=torch.bfloat16, device=DEV)
        st["v_sel"] = torch.empty_like(st["k_sel"])
    else:
        t = _tensors(case, seed)
        st["sel"] = _random_set(case, seed)
        rows = (st["sel"].long()[:, None] * c + torch.arange(c, device=DEV)).reshape(-1)
        short = (rows >= case["n"])[:, None, None]
        rows = rows.clamp(max=case["n"] - 1)
        st["k_sel"] = t["k"][rows].masked_fill(short, 0.0)
        st["v_sel"] = t["v"][rows].masked_fill(short, 0.0)
        st.update(q=t["q"], ks=t["ks"], vs=t["vs"], out=torch.empty_like(t["q"]))
        st["ws"] = _bytes(ckv.attn_workspace_bytes(dims, k))
    return st


def run(st):
    kind, dims, n_kept = st["kind"], st["dims"], st["n_kept"]
    if kind == "layer":
        t = st["layers"][0]
        st["ctx"].reprefill_layer(0, t["q"], t["ks"], t["vs"], t["k"], t["out"], k_prefix=t["k"],
                                  v_prefix=t["v"], chunk_scores=t["scores"], sel_idx=t["sel"])
        return {"scores": t["scores"], "sel": t["sel"], "out": t["out"]}
    if kind == "host":
        ctx, got = st["ctx"], []
        ctx.reset()  # a new request
        for i, t in enumerate(st["layers"]):
            stats = ctx.reprefill_layer(i, t["q"], t["ks"], t["vs"], t["k"], t["out"],
                                        chunk_scores=t["scores"], sel_idx=t["sel"])
            got.append({"scores": t["scores"], "sel": t["sel"], "out": t["out"],
                        "hits": stats["hits"], "misses": stats["misses"]})
        return got
    if kind == "score":
        ckv.score_chunks(dims, st["q"], st["k"], st["scores"], st["ws"])
        return st["scores"]
    if kind == "select":
        ckv.select_topk_chunks(st["scores"], st["m"], n_kept, st["sel"], st["ws"])
        return st["sel"]
    if kind == "gather":
        ckv.gather_chunks(dims, st["k"], st["v"], st["sel"], n_kept, st["k_sel"], st["v_sel"])
        return {"k": st["k_sel"], "v": st["v_sel"]}
    ckv.sparse_prefill_attn(dims, st["q"], st["k_sel"], st["v_sel"], st["sel"], n_kept,
                            st["ks"], st["vs"], st["out"], st["ws"])
    return st["out"]


def work(case):
    """Inputs read once and outputs written once, and the products of the definitions."""
    n, s, hq, hkv, d, c = (case[x] for x in ("n", "s", "hq", "hkv", "d", "c"))
    m, k = _sizes(case)
    eb = 4 if case["dtype"] == "f32" else 2
    kept = min(k * c, n)
    key_rows = hkv * d * eb  # bytes of one token's K (or V)
    qo = s * hq * d * eb
    score_flops = 2 * s * hq * d * n
    attn_flops = 4 * s * hq * d * (kept + (s + 1) / 2)
    kind = case["kind"]
    if kind == "score":
        return {"bytes": n * key_rows + qo + 8 * m, "flops": score_flops}
    if kind == "select":
        return {"bytes": 8 * m + 4 * k, "flops": 0}
    if kind == "gather":
        return {"bytes": 2 * 2 * kept * key_rows + 4 * k, "flops": 0}
    if kind == "attn":
        return {"bytes": 2 * (kept + s) * key_rows + 2 * qo + 4 * k, "flops": attn_flops}
    reads = n * key_rows + kept * key_rows + 2 * s * key_rows + qo  # K, kept V, suffix K/V, Q
    if kind == "host":
        reads += kept * key_rows  # the kept K come from the host store, not from the probe keys
    layers = case["layers"]
    return {"bytes": layers * (reads + qo + 8 * m + 4 * k),
            "flops": layers * (score_flops + attn_flops)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("select", "gather"):
        return "exact"
    if kind == "score":  # fp32 logits and per-chunk sums, fp64 sums across rows
        return {"rel": 4e-8, "max": 4e-7}
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 8e-2}


# ---- the definitions in 64 bits ----------------------------------------------

def _exact_scores(case, q, k):
    """A_j: softmax over the prefix of every (query, head), summed per chunk and over rows."""
    n, s, hq, hkv, d, c = (case[x] for x in ("n", "s", "hq", "hkv", "d", "c"))
    m, g = ckv.num_chunks(n, c), hq // hkv
    scale = 1.0 / math.sqrt(d)
    total = torch.zeros(m * c, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // n)
    for h in range(hkv):
        kt = k[:, h].double().t().contiguous()
        rows = q[:, h * g:(h + 1) * g].double().reshape(s * g, d) * scale
        for r in range(0, s * g, step):
            x = rows[r:r + step] @ kt
            x.sub_(x.amax(1, keepdim=True)).exp_()
            total[:n] += (x / x.sum(1, keepdim=True)).sum(0)
    return total.view(m, c).sum(1)


def _exact_attention(case, q, k, v, ks, vs, valid):
    """Attention over compact prefix rows k, v (those of `valid`) and the causal suffix."""
    s, hq, hkv, d = case["s"], case["hq"], case["hkv"], case["d"]
    g = hq // hkv
    scale = 1.0 / math.sqrt(d)
    k, v = k[valid], v[valid]
    p = k.shape[0]
    out = torch.empty((s, hq, d), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // (g * (p + s)))
    at = torch.arange(s, device=DEV)
    for h in range(hkv):
        kk = torch.cat((k[:, h], ks[:, h])).double().t().contiguous()
        vv = torch.cat((v[:, h], vs[:, h])).double()
        for t in range(0, s, step):
            rows = q[t:t + step, h * g:(h + 1) * g].double()
            b = rows.shape[0]
            x = (rows.reshape(b * g, d) * scale @ kk).view(b, g, p + s)
            hidden = at[None, :] > at[t:t + b, None]
            x[:, :, p:].masked_fill_(hidden[:, None, :], -math.inf)
            out[t:t + b, h * g:(h + 1) * g] = (torch.softmax(x, -1).view(b * g, p + s) @ vv).view(b, g, d)
    return out


def _top_k(scores, k):
    order = torch.sort(scores, descending=True, stable=True).indices[:k]
    return torch.sort(order).values


def exact(case, seed):
    kind = case["kind"]
    m, k = _sizes(case)
    c = case["c"]
    if kind == "score":
        t = _tensors(case, seed, names=("q", "k"))
        return _exact_scores(case, t["q"], t["k"])
    if kind == "select":
        return _top_k(_scores_like(case, seed), k).to(torch.int32)
    if kind == "gather":
        return None  # bytes are copied, nothing is computed
    got = []
    for layer in range(case["layers"]):
        t = _tensors(case, seed, layer)
        if kind == "attn":
            scores, sel = None, _random_set(case, seed)
        else:
            scores = _exact_scores(case, t["q"], t["k"])
            sel = _top_k(scores, k).to(torch.int32)
        rows = (sel.long()[:, None] * c + torch.arange(c, device=DEV)).reshape(-1)
        valid = rows < case["n"]
        rows = rows.clamp(max=case["n"] - 1)
        out = _exact_attention(case, t["q"], t["k"][rows], t["v"][rows], t["ks"], t["vs"], valid)
        if kind == "attn":
            return out
        got.append({"scores": scores, "sel": sel, "out": out})
        if kind == "host":
            got[-1].update(hits=None, misses=None)
    return got[0] if kind == "layer" else got
