"""The work that a program built on this library has it do, as measurable cases.

Four kinds of pass, each through the public binding with outputs and workspaces that the program
keeps between calls (as a serving loop does):

  attend    reform_chunk_attend_score: one layer's chunk of queries over [retained cache || chunk],
            with the eviction score (a prefill chunk) or without it (a generated token)
  compress  what follows a layer's attention: the selected heads' states go into the embedding
            store, the cache is evicted down to the budget, the kept keys are rotated to their new
            positions
  gather    reform_gather_topk: similarity search over the embedding store, top-k and its union
  recompute reform_gather_pooled, then reform_gather_rows of the selected tokens' inputs

Sizes are those of the repository's five workloads (paper_2506_01215_amd/synth.py), of its tests,
or generic.  `draw` gives more cases of the same ranges.
"""
import math

import torch
import torch.nn.functional as F

from paper_2506_01215_amd import binding

DEV = "cuda:0"
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}


def _attend(name, dtype, hq, hkv, d, cache, chunk, window=0, score=True, sinks=False):
    """window 0: every row of the chunk observes.  sinks: the first four keys draw most heads'
    attention, as they do in trained models (the eviction score then spans four decades)."""
    return {"name": name, "kind": "attend", "dtype": dtype, "hq": hq, "hkv": hkv, "d": d,
            "cache": cache, "chunk": chunk, "window": window, "score": score, "sinks": sinks}


def _compress(name, dtype, hkv, d, budget, chunk, heads, keep, rotary):
    """heads: selected heads whose states are saved; keep: first and last slots always kept."""
    return {"name": name, "kind": "compress", "dtype": dtype, "hkv": hkv, "d": d, "budget": budget,
            "chunk": chunk, "heads": heads, "keep": keep, "rotary": rotary}


def _gather(name, dtype, n, dim, queries, k, radius, keep=0):
    return {"name": name, "kind": "gather", "dtype": dtype, "n": n, "dim": dim, "queries": queries,
            "k": k, "radius": radius, "keep": keep}


def _recompute(name, dtype, n, dim, queries, budget, window, keep, hidden):
    return {"name": name, "kind": "recompute", "dtype": dtype, "n": n, "dim": dim,
            "queries": queries, "budget": budget, "window": window, "keep": keep, "hidden": hidden}


def listed():
    return [
        # the smallest stream: a verification-sized fp32 layer, chunks of 128 (workload 1)
        _attend("attend_f32_small", "f32", 4, 4, 64, 256, 128),
        # the ragged end of a prompt: 17 rows over a full 4096-slot cache, one KV head per query
        # head (workload 5's last chunk)
        _attend("attend_tail_17", "bf16", 8, 8, 128, 4096, 17, sinks=True),
        # one generated token over a 16k recomputed cache and what was generated so far: attention
        # alone, once per layer and token
        _attend("attend_token_16k", "bf16", 32, 8, 128, 16640, 1, score=False, sinks=True),
        # the compressor as the paper's experiments set it (128 observing rows), an odd chunk,
        # 64-wide heads, three query heads per KV head
        _attend("attend_window_3001", "bf16", 24, 8, 64, 8192, 3001, window=128, sinks=True),
        # a 128k-token layer in chunks of 8192 (workload 2)
        _attend("attend_8k", "bf16", 32, 8, 128, 8192, 8192),
        # a 1M-token layer in chunks of 32768 with a full cache (workload 3): the headline step
        _attend("attend_32k", "bf16", 32, 8, 128, 32768, 32768),
        # compression after that ragged end: 17 of 4113 slots go
        _compress("compress_tail_17", "bf16", 8, 128, 4096, 17, 4, 0, 128),
        # compression after a full chunk of the 1M stream, first and last 256 slots protected
        _compress("compress_32k", "bf16", 8, 128, 32768, 32768, 4, 256, 128),
        # similarity search over a 2k prompt, fp32 (workload 1)
        _gather("gather_f32_2k", "f32", 2048, 256, 1, 128, 0),
        # over a 128k prompt, one query embedding (workload 2)
        _gather("gather_128k", "bf16", 131072, 1024, 1, 4096, 0),
        # over a 1M prompt, 16 query tokens and their neighbourhoods (workload 4)
        _gather("gather_1m", "bf16", 1048576, 2048, 16, 16384, 8),
        # the paper's own selection over a 256k prompt for a question of 37 tokens, then the inputs
        # of the selected tokens
        _recompute("recompute_256k", "bf16", 262144, 1024, 37, 8192, 129, 256, 4096),
    ]


def _log(rng, lo, hi):
    """An integer whose logarithm is spread evenly over [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attend", "attend", "attend", "attend", "token", "f32", "compress",
                       "compress", "gather", "gather", "recompute"])
    hq, hkv = rng.choice([(32, 8), (32, 8), (24, 8), (8, 8), (16, 4), (14, 2)])
    d = rng.choice([128, 128, 128, 64])
    if kind == "attend":
        chunk = _log(rng, 8, 16384)
        cache = rng.choice([0, _log(rng, 512, 32768), _log(rng, 512, 32768)])
        window = min(128, chunk) if rng.random() < 0.4 else 0
        c = _attend("", "bf16", hq, hkv, d, cache, chunk, window, True, rng.random() < 0.5)
    elif kind == "token":
        c = _attend("", "bf16", hq, hkv, d, _log(rng, 1024, 65536), rng.choice([1, 1, 1, 2, 4]),
                    score=False, sinks=True)
    elif kind == "f32":
        h = rng.choice([(4, 4), (8, 4), (8, 2)])
        c = _attend("", "f32", h[0], h[1], rng.choice([64, 64, 32, 128]), _log(rng, 64, 1024),
                    _log(rng, 16, 512))
    elif kind == "compress":
        budget = _log(rng, 512, 32768)
        keep = min(256, budget // 4) if rng.random() < 0.5 else 0
        c = _compress("", "bf16", hkv, d, budget, _log(rng, 16, 32768), rng.choice([1, 2, 4]), keep, d)
    elif kind == "gather":
        if rng.random() < 0.25:
            n = _log(rng, 500, 16384)
            c = _gather("", "f32", n, rng.choice([64, 128, 256, 512]), rng.choice([1, 4, 16]),
                        max(1, n // 16), rng.choice([0, 8]))
        else:
            n = _log(rng, 4000, 1000000)
            c = _gather("", "bf16", n, 128 * rng.randint(2, 16), rng.choice([1, 1, 5, 16, 16, 23]),
                        max(1, n // rng.choice([8, 32, 64])), rng.choice([0, 8, 64]), rng.choice([0, 256]))
    else:
        n = _log(rng, 8000, 600000)
        budget = max(64, min(16384, n // rng.choice([4, 16])))
        c = _recompute("", "bf16", n, 128 * rng.randint(2, 16), rng.randint(1, 64), budget,
                       rng.choice([129, 129, 33]), min(256, budget // 4), rng.choice([2048, 4096]))
    del c["name"]
    return c


def _workspace(nbytes):
    return torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)


def _states(gen, hq, hkv, d, n, chunk, sinks):
    """Q of the last `chunk` of n tokens, K and V of all of them.  Half of a query's and a key's
    energy lies in 16 directions that the heads share and is common to one token, so attention
    concentrates; key norms vary from token to token."""
    def randn(*shape):
        return torch.randn(shape, generator=gen, device=DEV)

    basis = torch.linalg.qr(randn(d, 16))[0].t()
    shared = (randn(n, 16) @ basis) * math.sqrt(d / 32.0)
    q = randn(hq, chunk, d).mul_(math.sqrt(0.5)).add_(shared[n - chunk:])
    k = randn(hkv, n, d).mul_(math.sqrt(0.5)).add_(shared)
    k *= torch.exp(0.25 * randn(1, n, 1))
    v = randn(hkv, n, d)
    if sinks:
        u = F.normalize(randn(hkv, 1, d), dim=-1)
        q += 2.0 * u.repeat_interleave(hq // hkv, dim=0)
        s = min(4, n)
        k[:, :s] = 3.0 * math.sqrt(d) * u
    return q, k, v


def _prepare_attend(c, gen):
    dt, n = DTYPE[c["dtype"]], c["cache"] + c["chunk"]
    q, k, v = _states(gen, c["hq"], c["hkv"], c["d"], n, c["chunk"], c["sinks"])
    s = {"q": q.to(dt), "k": k.to(dt).contiguous(), "v": v.to(dt).contiguous()}
    s["out"] = torch.zeros_like(s["q"])
    s["lse"] = torch.zeros(q.shape[:2], dtype=torch.float32, device=DEV)
    s["score"] = torch.zeros(k.shape[:2], dtype=torch.float32, device=DEV) if c["score"] else None
    s["scale"] = 1.0 / math.sqrt(c["d"])
    desc = binding.attn_desc(s["q"], s["k"], s["out"], c["cache"], s["scale"], c["window"])
    s["ws"] = _workspace(binding.attend_workspace_bytes(desc))
    return s


def _prepare_compress(c, gen):
    dt, h, d, budget, chunk = DTYPE[c["dtype"]], c["hkv"], c["d"], c["budget"], c["chunk"]
    n = budget + chunk
    s = {"k": torch.randn((h, n, d), generator=gen, device=DEV).to(dt),
         "v": torch.randn((h, n, d), generator=gen, device=DEV).to(dt),
         "q": torch.randn((c["heads"], chunk, d), generator=gen, device=DEV).to(dt)}
    # column sums of attention: the cache is seen by every row of the chunk, chunk row i by the
    # rows from i on; heavy tails over the tokens
    seen = torch.full((n,), float(chunk), device=DEV)
    seen[budget:] = torch.arange(chunk, 0, -1, device=DEV, dtype=torch.float32)
    s["new_score"] = torch.exp(torch.randn((h, n), generator=gen, device=DEV)) * (seen / n)
    s["score"] = torch.zeros_like(s["new_score"])
    s["pos"] = torch.arange(n, dtype=torch.int32, device=DEV).repeat(h, 1)
    s["kept"] = torch.zeros((h, budget), dtype=torch.int32, device=DEV)
    s["emb"] = torch.zeros((chunk, 2 * c["heads"] * d), dtype=dt, device=DEV)
    s["ws"] = _workspace(binding.evict_workspace_bytes(
        binding.evict_desc(s["k"], n, budget, c["keep"], c["keep"])))
    return s


def _store(c, gen):
    """Embedding store and query embeddings: 128-wide head segments of unit length, with passages
    that lie close to the queries."""
    dt, n, dim = DTYPE[c["dtype"]], c["n"], c["dim"]
    seg = min(128, dim)
    qry = torch.randn((c["queries"], dim), generator=gen, device=DEV)
    near = torch.randint(0, n, (16,), generator=gen, device=DEV)
    hit = (near.view(-1, 1) + torch.arange(32, device=DEV)).clamp_(max=n - 1).view(-1)
    emb = torch.empty((n, dim), dtype=dt, device=DEV)
    for r in range(0, n, 65536):
        x = torch.randn((min(65536, n - r), dim), generator=gen, device=DEV)
        inside = hit[(hit >= r) & (hit < r + x.shape[0])] - r
        x[inside] += 0.3 * qry[inside % qry.shape[0]]
        emb[r:r + x.shape[0]] = F.normalize(x.view(-1, seg), dim=-1).view(x.shape).to(dt)
    return emb, F.normalize(qry.view(-1, seg), dim=-1).view(qry.shape).to(dt)


def _prepare_gather(c, gen):
    emb, qry = _store(c, gen)
    i32 = dict(dtype=torch.int32, device=DEV)
    desc = binding.gather_desc(emb, qry, c["k"], c["radius"], c["keep"], c["keep"])
    return {"emb": emb, "qry": qry, "topk_idx": torch.zeros((c["queries"], c["k"]), **i32),
            "topk_score": torch.zeros((c["queries"], c["k"]), dtype=torch.float32, device=DEV),
            "union_idx": torch.zeros(c["n"], **i32), "union_count": torch.zeros(1, **i32),
            "ws": _workspace(binding.gather_workspace_bytes(desc))}


def _prepare_recompute(c, gen):
    emb, qry = _store(c, gen)
    desc = binding.pooled_desc(emb, qry, c["budget"], c["window"], c["keep"], c["keep"])
    table = torch.randn((c["n"], c["hidden"]), generator=gen, device=DEV, dtype=DTYPE[c["dtype"]])
    return {"emb": emb, "qry": qry, "table": table,
            "sel": torch.zeros(c["budget"], dtype=torch.int32, device=DEV),
            "pooled": torch.zeros(c["n"], dtype=torch.float32, device=DEV),
            "rows": torch.zeros((c["budget"], c["hidden"]), dtype=table.dtype, device=DEV),
            "ws": _workspace(binding.pooled_workspace_bytes(desc))}


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    make = {"attend": _prepare_attend, "compress": _prepare_compress, "gather": _prepare_gather,
            "recompute": _prepare_recompute}[case["kind"]]
    return dict(make(case, gen), case=dict(case))


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "attend":
        out, lse, score = binding.reform_chunk_attend_score(
            s["q"], s["k"], s["v"], c["cache"], s["scale"], obs_window=c["window"], out=s["out"],
            lse=s["lse"], score=s["score"], want_score=c["score"], workspace=s["ws"])
        return {"out": out, "lse": lse, "score": score}
    if c["kind"] == "compress":
        n, keep = c["budget"] + c["chunk"], c["keep"]
        s["score"].copy_(s["new_score"])          # stands for the attention call that wrote them
        binding.reform_embed_save_selected(s["q"], s["emb"], 0, c["heads"] * c["d"])
        binding.reform_evict_topk_compact(s["k"], s["v"], s["score"], n, c["budget"], keep, keep,
                                          pos=s["pos"], kept_idx=s["kept"], workspace=s["ws"])
        binding.reform_rerotate_keys(s["k"], s["kept"], c["budget"], 1e6, c["rotary"])
        return {x: s[x] for x in ("emb", "k", "v", "score", "pos", "kept")}
    if c["kind"] == "gather":
        idx, val, union, count = binding.reform_gather_topk(
            s["emb"], s["qry"], c["k"], c["radius"], c["keep"], c["keep"], topk_idx=s["topk_idx"],
            topk_score=s["topk_score"], union_idx=s["union_idx"], union_count=s["union_count"],
            workspace=s["ws"])
        return {"topk_idx": idx, "topk_score": val, "union_idx": union, "union_count": count}
    sel, pooled = binding.reform_gather_pooled(
        s["emb"], s["qry"], c["budget"], c["window"], c["keep"], c["keep"], sel_idx=s["sel"],
        pooled=s["pooled"], workspace=s["ws"])
    rows = binding.reform_gather_rows(s["table"], sel, out=s["rows"])
    return {"sel": sel, "pooled": pooled, "rows": rows}


def work(case):
    c, e = case, SIZE[case["dtype"]]
    if c["kind"] == "attend":
        m, ct, d = c["cache"], c["chunk"], c["d"]
        pairs = ct * m + ct * (ct + 1) / 2.0
        flops = 4.0 * d * c["hq"] * pairs                 # Q.K and P.V of the visible pairs
        nbytes = e * d * (2.0 * c["hkv"] * (m + ct) + 2.0 * c["hq"] * ct) + 4.0 * c["hq"] * ct
        if c["score"]:
            w = c["window"] or ct                         # the score needs the final normaliser:
            seen = w * m + w * (ct - w) + w * (w + 1) / 2.0   # Q.K of the observing rows again
            flops += 2.0 * d * c["hq"] * seen
            nbytes += 4.0 * c["hkv"] * (m + ct)
        return {"bytes": nbytes, "flops": flops}
    if c["kind"] == "compress":
        h, d, b, n = c["hkv"], c["d"], c["budget"], c["budget"] + c["chunk"]
        # `chunk` slots go, at places spread over the cache: every row behind the first one moves
        moved = b * c["chunk"] / (c["chunk"] + 1.0)
        nbytes = 4.0 * h * n + 4.0 * h * b                # scores read, kept slots written
        nbytes += h * moved * (4.0 * e * d + 16.0)        # K, V, score and pos of the moved rows
        nbytes += 2.0 * e * c["heads"] * c["chunk"] * d   # saved states
        return {"bytes": nbytes, "flops": 3.0 * h * moved * d}
    nq, n, dim = c["queries"], c["n"], c["dim"]
    nbytes, flops = float(e) * (n + nq) * dim, 2.0 * nq * n * dim
    if c["kind"] == "gather":
        hits = min(float(n), nq * c["k"] * (1.0 + 2.0 * c["radius"]))
        return {"bytes": nbytes + 8.0 * nq * c["k"] + 4.0 * min(hits, n / 2.0), "flops": flops}
    return {"bytes": nbytes + 4.0 * n + 4.0 * c["budget"] + 2.0 * e * c["budget"] * c["hidden"],
            "flops": flops}


def tolerance(case):
    if case["kind"] == "attend":
        # against the same sums in 64 bits, measured on the small listed cases: bf16 2.1e-3
        # (largest 1.9e-2; the outputs and the probabilities of P.V are rounded to bf16, the
        # latter relative to whichever running maximum an implementation's order gives); fp32
        # 4e-7 (largest 5e-6, for a few hundred keys)
        return {"rel": 1e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 5e-5}
    if case["kind"] == "compress":
        # selections and moves are exact; saved states and rotated keys are rounded to bf16
        return {"rel": 5e-3, "max": 0.1}
    # similarities are 32-bit sums of up to 2048 products: 2e-7 (largest 8e-7) against 64 bits;
    # a selection may swap neighbours in value, which shifts the indices between them
    return {"rel": 2e-6, "max": 1e-5, "differ": 0.01}
