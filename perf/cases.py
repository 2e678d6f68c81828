"""Timed cases of the prefix-cached attention path, through its public entry points.

A case is one attention layer's work on one batch, in one of five forms:

    prefill  K/V append (optionally with RoPE) of the uncached suffix rows, then
             attention of the suffix queries over cached prefix + suffix; split
             at the shared prefix where the library's rule prefers that
    chunk    the same prefill cut into scheduler steps of at most ``budget`` new
             tokens, captured once (ChunkGraph) and replayed
    decode   append of the newest ``rows`` tokens of every request, then their
             attention over the whole context
    serve    a whole call: host prefix match, metadata upload, append, attention
    steps    the chunked prefill issued step by step (no captured graph)

Prompts are ``shared`` common tokens (the instruction and leading
demonstrations), ``own`` cached tokens of each request's own, and ``new``
uncached ones; lengths spread evenly over [lo, hi].  Head shapes and lengths
are those of the repository's workloads and shape tests (`workload.SPECS`).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2507_08523_amd import ilpc, pipeline

BLOCK = ilpc.BLOCK
ROPE_BASE = 500000.0


def _case(kind, heads, b, shared, own, new, q_std=1.0, rope=False, rows=1, budget=0, name=None):
    hq, hkv, d = heads
    c = {"kind": kind, "hq": hq, "hkv": hkv, "d": d, "b": b, "shared": shared, "own_lo": own[0],
         "own_hi": own[1], "new_lo": new[0], "new_hi": new[1], "q_std": q_std, "rope": rope, "rows": rows,
         "budget": budget}
    if name:
        c["name"] = name
    return c


LLAMA, QWEN, LARGE, TINY = (32, 8, 128), (28, 4, 128), (64, 8, 128), (4, 1, 64)


def listed():
    return [
        # the smallest batch of the repository: launches and latency only
        _case("prefill", TINY, 4, 64, (0, 0), (32, 32), name="prefill_tiny"),
        # one interactive request: a long cached prompt and a short new log line
        _case("prefill", LARGE, 1, 0, (2048, 2048), (64, 64), name="prefill_one_request"),
        # a serving step end to end on the Llama-3-8B-shaped layer: 64 prompts of
        # 604 tokens, about half cached, K and Q rotated in the append
        _case("serve", LLAMA, 64, 256, (0, 96), (300, 300), rope=True, name="serve_llama8b"),
        # ragged prompts on the Qwen2.5-7B-shaped layer (head group of 7)
        _case("prefill", QWEN, 256, 512, (0, 128), (520, 720), q_std=128 ** -0.5, name="prefill_qwen7b"),
        # nothing cached: the hit-rate sweep's 0% point
        _case("prefill", LLAMA, 128, 0, (0, 0), (1024, 1024), name="prefill_uncached"),
        # everything but the query log cached and shared: the sweep's 100% point,
        # which the library's rule sends through the shared-prefix split
        _case("prefill", LLAMA, 128, 976, (0, 0), (48, 48), name="prefill_shared_split"),
        # every prompt's own long prefix cached, short suffixes
        _case("prefill", LARGE, 512, 0, (2048, 2048), (64, 64), name="prefill_own_prefix"),
        # the largest shapes (64 q heads, 2112-token prompts), almost nothing cached
        _case("prefill", LARGE, 128, 128, (0, 0), (1984, 1984), name="prefill_large"),
        # chunked prefill under a 1024-token scheduler budget, replayed as a graph
        _case("chunk", LLAMA, 64, 256, (0, 96), (300, 300), budget=1024, name="chunk_llama8b"),
        # decode of a handful of requests (each pair's keys split over several waves)
        _case("decode", LARGE, 4, 0, (2100, 2130), (1, 1), name="decode_few"),
        # decode of a batch that shares its prompt's prefix
        _case("decode", LLAMA, 128, 976, (32, 64), (1, 1), name="decode_shared"),
        # decode of the largest batch: 512 contexts of about 2.1 K tokens
        _case("decode", LARGE, 512, 0, (2100, 2140), (1, 1), name="decode_large"),
    ]


# head shapes of the workloads and of the shape tests (groups of 1 to 16, both head sizes)
_HEADS = [LLAMA, LLAMA, QWEN, LARGE, TINY, (8, 8, 128), (16, 2, 64), (20, 4, 128), (32, 2, 128), (12, 4, 64)]
_MOST_FLOPS, _MOST_BYTES = 3.0e12, 6.0e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "serve", "chunk", "steps"])
        heads = rng.choice(_HEADS)
        b = _log_int(rng, 1, 512)
        shared = rng.choice([0, 16 * _log_int(rng, 1, 96)])
        own_hi = rng.choice([0, _log_int(rng, 16, 4096)])
        own = (rng.randint(own_hi // 2, own_hi), own_hi)
        q_std = rng.choice([heads[2] ** -0.5, 1.0, 1.0, 3.0])
        rope = rng.random() < 0.4
        if kind == "decode":
            rows = rng.choice([1, 1, 1, 2, 3])
            if rows * (heads[0] // heads[1]) > 32:
                rows = 1
            if shared + own[0] < 16:
                continue
            c = _case(kind, heads, b, shared, own, (rows, rows), q_std, rope, rows)
        else:
            new_hi = _log_int(rng, 1, 2112)
            budget = _log_int(rng, 128, 8192) if kind in ("chunk", "steps") else 0
            c = _case(kind, heads, b, shared, own, (rng.randint(max(1, new_hi // 2), new_hi), new_hi), q_std,
                      rope, 1, budget)
            if budget and sum(_lens(c)[1]) > 24 * budget:
                continue
        w = work(c)
        if w["flops"] <= _MOST_FLOPS and w["bytes"] <= _MOST_BYTES:
            return c


# -- shapes -------------------------------------------------------------------

def _lens(case):
    """(own cached tokens, new tokens) of every request, the same for every seed."""
    b = case["b"]
    rng = np.random.default_rng([b, case["own_hi"], case["new_hi"]])

    def spread(lo, hi):
        return rng.permutation(np.round(np.linspace(lo, hi, b)).astype(np.int64))

    return spread(case["own_lo"], case["own_hi"]), spread(case["new_lo"], case["new_hi"])


def _cached(case, own, new):
    """Cached length of every request: whole blocks only, and at least one token recomputed
    (decode: the whole context is there already)."""
    ctx = case["shared"] + own
    return ctx if case["kind"] == "decode" else ctx // BLOCK * BLOCK


def _prompt_lens(case):
    own, new = _lens(case)
    P = _cached(case, own, new)
    L = case["shared"] + own + new
    return P, L


def work(case):
    P, L = (x.astype(np.float64) for x in _prompt_lens(case))
    S = L - P
    kv, qo = 4.0 * case["hkv"] * case["d"], 2.0 * case["hq"] * case["d"]
    pairs = float(np.sum(S * P + S * (S + 1) / 2))
    # the shared prefix counts once; a request's own cached tokens and its new
    # K/V rows are read once, the new rows are written to the pools, Q is read
    # and the output (with RoPE also the rotated Q) written
    whole = case["shared"] // BLOCK * BLOCK
    cached = float(np.sum(P - np.minimum(P, whole))) + whole
    n = float(S.sum())
    return {"bytes": kv * cached + 2 * kv * n + (3 if case["rope"] else 2) * qo * n,
            "flops": 4.0 * case["hq"] * case["d"] * pairs}


def tolerance(case):
    # bf16 outputs and bf16 softmax probabilities (fp32 sums); with RoPE also
    # bf16 rotated Q and K, and fp32 angles at positions of a few thousand
    return {"rel": 0.012, "max": 0.3, "differ": 0.0}


# -- inputs -------------------------------------------------------------------

def prepare(case, seed):
    own, new = _lens(case)
    P, L = _prompt_lens(case)
    b, hq, hkv, d = case["b"], case["hq"], case["hkv"], case["d"]
    rng = np.random.default_rng([seed, 1])
    shared = rng.integers(0, 32000, case["shared"], dtype=np.int32)
    prompts = []
    for r in range(b):
        t = rng.integers(0, 32000, int(own[r] + new[r]), dtype=np.int32)
        t[0] = 32000 + r  # sharing ends with the shared tokens
        prompts.append(np.concatenate([shared, t]))
    decode = case["kind"] == "decode"
    n_warm = [int(x) // BLOCK * BLOCK for x in (L - new if decode else P)]
    blocks = len(shared) // BLOCK + sum(-(-int(x) // BLOCK) for x in L) + 8
    blocks += sum(max(0, n - len(shared)) // BLOCK + 2 for n in n_warm)
    max_blocks = -(-int(L.max()) // BLOCK)
    log2cap = max(10, int(math.ceil(math.log2(blocks * 8 / 7 + 1))) + 1)
    pc = pipeline.PagedPrefixCache(hkv, d, blocks, max_blocks, b, log2cap)
    # the cached part of the batch: the shared prefix first, then each request's own
    if len(shared) >= BLOCK:
        pc.match([shared])
    warm = [p[:n] for p, n in zip(prompts, n_warm) if n > len(shared) // BLOCK * BLOCK]
    if warm:
        pc.match(warm)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def randn(*shape, std=1.0):
        x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)
        return x if std == 1.0 else x.mul_(std)

    pc.k_pool.copy_(randn(*pc.k_pool.shape))
    pc.v_pool.copy_(randn(*pc.v_pool.shape))
    n = int((L - P).sum())
    st = {"case": case, "pc": pc, "P": P, "L": L, "scale": 1.0 / math.sqrt(d),
          "q": randn(n, hq, d, std=case["q_std"]), "k_new": randn(n, hkv, d), "v_new": randn(n, hkv, d),
          "out": torch.zeros(n, hq, d, dtype=torch.bfloat16, device="cuda"), "inv_freq": None, "q_rot": None}
    if case["rope"]:
        st["inv_freq"] = torch.from_numpy(pipeline.rope_inv_freq(d, ROPE_BASE)).cuda()
        st["q_rot"] = torch.zeros_like(st["q"])
    cu = np.zeros(b + 1, np.int32)
    cu[1:] = np.cumsum(L - P)
    st["cu"] = cu
    st["packed"] = (np.concatenate(prompts), np.concatenate([[0], np.cumsum(L)]).astype(np.int32))
    mark = pc.cache.checkpoint()
    st["cached"], st["tables"] = pc.match(packed=st["packed"])
    if not decode and not np.array_equal(st["cached"], P):
        raise RuntimeError("the cached lengths are not the case's")
    if case["kind"] == "serve":
        pc.cache.rollback(mark)
        return st
    if case["kind"] == "chunk":
        st["graph"] = pipeline.ChunkGraph(pc, P.astype(np.int32), st["tables"], L.astype(np.int32), st["q"],
                                          st["k_new"], st["v_new"], st["out"], st["scale"], case["budget"],
                                          st["inv_freq"], st["q_rot"])
        return st
    if case["kind"] == "steps":
        return st
    st["batch"] = pc.upload(st["tables"], cu, L.astype(np.int32), P.astype(np.int32))
    st["split"] = 0
    if not decode:
        shared_len = pipeline.shared_prefix_len(st["cached"], st["tables"])
        if pipeline.prefer_shared_split(L, st["batch"].max_q_len, hq, hkv, shared_len):
            st["split"] = shared_len
            st["ws"] = pc.cascade_workspace(st["batch"], hq)
    return st


# -- one pass -----------------------------------------------------------------

def _append(st, batch):
    if st["inv_freq"] is None:
        st["pc"].append(batch, st["k_new"], st["v_new"])
        return st["q"]
    st["pc"].append_rope(batch, st["k_new"], st["v_new"], st["inv_freq"], st["q"], st["q_rot"])
    return st["q_rot"]


def _outputs(st, **more):
    res = {"out": st["out"], "k_pool": st["pc"].k_pool, "v_pool": st["pc"].v_pool, **more}
    if st["q_rot"] is not None:
        res["q_rot"] = st["q_rot"]
    return res


def run(st):
    kind, pc = st["case"]["kind"], st["pc"]
    if kind == "chunk":
        st["graph"].replay()
        return _outputs(st)
    if kind == "steps":
        pc.prefill_chunked(st["cached"], st["tables"], st["L"], st["q"], st["k_new"], st["v_new"], st["out"],
                           st["scale"], st["case"]["budget"], inv_freq=st["inv_freq"], q_rot=st["q_rot"])
        return _outputs(st)
    if kind == "serve":
        mark = pc.cache.checkpoint()
        cached, tables = pc.match(packed=st["packed"])
        batch = pc.upload_prefill(cached, tables, st["L"])
        pc.cache.rollback(mark)  # the next pass serves the same batch again
        pc.attend(batch, _append(st, batch), st["out"], st["scale"])
        return _outputs(st, cached=cached, tables=tables)
    q = _append(st, st["batch"])
    if st["split"]:
        pc.attend_cascade(st["batch"], q, st["out"], st["scale"], st["split"], st["ws"])
    else:
        pc.attend(st["batch"], q, st["out"], st["scale"])
    return _outputs(st)


# -- the same in 64 bits --------------------------------------------------------

def _rotate(x, pos, inv_freq):
    """Rotate-half RoPE of rows x [n, H, D] (float64) at positions pos [n]."""
    half = x.shape[-1] // 2
    a = pos[:, None].double() * inv_freq[None, :].double()
    c, s = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def exact(case, seed):
    st = prepare(case, seed)
    pc, cu = st["pc"], st["cu"]
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    g = hq // hkv
    # prepare() may have run the path once (a captured graph); the rows it
    # wrote are written again below
    k_pool, v_pool = pc.k_pool.double(), pc.v_pool.double()
    out = torch.zeros(st["out"].shape, dtype=torch.float64, device="cuda")
    q_rot = torch.zeros_like(out) if case["rope"] else None
    tables = torch.from_numpy(st["tables"]).cuda().long()
    for r in range(case["b"]):
        P, L = int(st["P"][r]), int(st["L"][r])
        rows = slice(int(cu[r]), int(cu[r + 1]))
        pos = torch.arange(P, L, device="cuda")
        q, k, v = (st[n][rows].double() for n in ("q", "k_new", "v_new"))
        if case["rope"]:
            q, k = _rotate(q, pos, st["inv_freq"]), _rotate(k, pos, st["inv_freq"])
            q_rot[rows] = q
        phys, slot = tables[r][pos // BLOCK], pos % BLOCK
        k_pool[phys, :, slot, :] = k
        v_pool[phys, :, :, slot] = v
        at = torch.arange(L, device="cuda")
        p, s = tables[r][at // BLOCK], at % BLOCK
        kk = k_pool[p, :, s, :].transpose(0, 1).contiguous()        # [Hkv, L, D]
        vv = v_pool[p, :, :, s].transpose(0, 1).contiguous()
        qq = q.reshape(L - P, hkv, g, d).permute(1, 2, 0, 3).reshape(hkv, g * (L - P), d).contiguous()
        sc = torch.bmm(qq, kk.transpose(1, 2).contiguous()).mul_(st["scale"])
        sc.view(hkv, g, L - P, L).masked_fill_(at[None, :] > pos[:, None], -math.inf)
        o = torch.bmm(torch.softmax(sc, dim=-1), vv)
        out[rows] = o.reshape(hkv, g, L - P, d).permute(2, 0, 1, 3).reshape(L - P, hq, d)
        del sc, o
    res = {"out": out, "k_pool": k_pool, "v_pool": v_pool}
    if case["rope"]:
        res["q_rot"] = q_rot
    if case["kind"] == "serve":
        res["cached"] = res["tables"] = None
    return res
