"""The calls whose speed matters to a user of this library, as cases that can be timed and compared.

A case is one pass over one attention layer through `paper_2412_06198_amd.Session`, on synthetic
inputs made on the GPU from a seed: N(0,1) queries, keys and values with the attention structure the
method looks for planted in them (sink keys, vertical columns, diagonals, local windows, hot
blocks), so that the pattern rule meets heads of every kind.

    layer     scores, index and sparse attention of a prompt: what a prefill runs per layer
    dense     the attention call on an index that keeps every key (prompts below the sparse crossover)
    estimate  the scores alone
    index     the index alone, from given scores
    decode    one generated token over the prompt's index
    search    the offline per-head pattern search
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2412_06198_amd as sa

D = 128        # head dimension of every layer this library accepts
BETA = 3.0     # planted logit bias
PLANT_LO = 96  # dims below carry the noise, dims from here on the plants
CODE_LO = 100  # dims of the block codes


def _case(name, kind, hq, hkv, n, block, keep, mix, **more):
    c = {"kind": kind, "hq": hq, "hkv": hkv, "n": n, "block": block, "keep": keep, "mix": mix, "window": 64}
    c.update(more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a short prompt without grouped heads, where launches count
        _case("layer-4k", "layer", 4, 4, 4096, 64, 0.10, "slash"),
        # a prompt that ends in the middle of a 128-row block, index in one call, both selection options
        _case("layer-10k-ragged", "layer", 32, 8, 10304, 64, 0.18, "tiib", one_call=True, block_select=1,
              diagonal_select=1),
        # the benchmark's grouped-head layer (32 query, 8 key/value heads) at 16K, 32K and 128K tokens
        _case("layer-16k", "layer", 32, 8, 16384, 64, 0.125, "mod3"),
        _case("layer-32k", "layer", 32, 8, 32768, 64, 0.06, "tiib"),
        # the one-call form that computes the block map only for the heads that need it
        _case("layer-64k", "layer", 32, 8, 65536, 128, 0.04, "tiib", one_call=True, lazy=True),
        _case("layer-128k", "layer", 32, 8, 131072, 128, 0.03, "tiib"),
        # every key kept: plain causal attention, the baseline of the sparse path
        _case("dense-16k", "dense", 32, 8, 16384, 64, 1.0, "none"),
        # the two index stages by themselves, as a program calls them that keeps scores and index apart
        _case("estimate-32k", "estimate", 32, 8, 32768, 64, 0.06, "tiib"),
        _case("index-64k", "index", 32, 8, 65536, 128, 0.04, "tiib"),
        # a generated token after a short and after a long prompt
        _case("decode-4k", "decode", 8, 2, 4096, 64, 0.10, "slash", generated=1),
        _case("decode-128k", "decode", 32, 8, 131072, 128, 0.03, "tiib", generated=700),
        # the offline search over the heads of a small calibration prompt
        _case("search-4k", "search", 8, 2, 4096, 64, 0.30, "tiib"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer"] * 5 + ["dense", "estimate", "index", "decode", "decode", "search"])
    top = {"dense": 16384, "search": 4096}.get(kind, 131072)
    block = rng.choice([64, 128])
    n = min(top, max(8, _log_int(rng, 1024, top) // block) * block)
    heads = [(4, 4), (8, 8), (8, 2), (6, 2), (8, 1)]
    if kind != "search":
        heads += [(16, 4), (32, 8), (32, 8), (24, 3)]
    hq, hkv = rng.choice(heads)
    # what a query keeps grows slowly with the prompt: some 400 to 4000 keys
    keep = 1.0 if kind == "dense" else round(min(0.5, max(0.01, _log_int(rng, 400, min(4000, n)) / n)), 4)
    if kind == "search":
        keep = round(rng.uniform(0.05, 0.30), 3)
    c = _case("", kind, hq, hkv, n, block, keep, "none" if kind == "dense" else rng.choice(["tiib", "tiib", "mod3", "slash", "none"]))
    if kind in ("layer", "estimate", "index"):
        c["window"] = rng.choice([64, 64, 64, 32, 17])
    if kind == "layer":
        c["one_call"] = rng.random() < 0.5
        c["lazy"] = c["one_call"] and rng.random() < 0.5
        c["override"] = rng.random() < 0.25
    if kind in ("layer", "index"):
        c["block_select"] = rng.choice([0, 0, 0, 1, 2])
        c["diagonal_select"] = rng.choice([0, 0, 0, 1])
    if kind == "decode":
        c["generated"] = _log_int(rng, 1, 2000)
    return c


# ------------------------------------------------------------------------------------------- inputs
def _patterns(case):
    """The structure planted in each query head: a pattern of the library, or -1 for plain noise."""
    t, i, b = sa.SA_TRIANGULAR, sa.SA_INTERVAL_SLASH, sa.SA_BLOCK_CLUSTER
    cycle = {"tiib": [t, i, i, b], "mod3": [t, i, b], "slash": [i], "none": [-1]}[case["mix"]]
    return [cycle[h % len(cycle)] for h in range(case["hq"])]


def _noise(gen, *shape):
    """N(0,1) in fp32, the dims that carry plants cleared."""
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    x[..., PLANT_LO:] = 0.0
    return x


def _inputs(case, seed, rows=None):
    """Q [hq, n, 128], K and V [hkv, rows or n, 128] in bf16."""
    hq, hkv, n, block, w = case["hq"], case["hkv"], case["n"], case["block"], case["window"]
    rows = rows or n
    g = hq // hkv
    gen = torch.Generator(device="cuda").manual_seed(seed)
    host = np.random.RandomState(seed % (1 << 32))
    a = math.sqrt(BETA * math.sqrt(D))
    gain = BETA * math.sqrt(D) / PLANT_LO
    pats = _patterns(case)
    ncol, noff, nhot = (32, 16, 128) if n >= 65536 else (16, 8, 32)
    half = 512
    nhalf, nblk = -(-n // half), -(-n // block)
    idx_half = torch.arange(n, device="cuda") // half
    idx_blk = torch.arange(n, device="cuda") // block

    def codes(k):
        u = host.standard_normal((k, D - CODE_LO)).astype(np.float32)
        return u / np.linalg.norm(u, axis=1, keepdims=True)

    Q = torch.empty((hq, n, D), dtype=torch.bfloat16, device="cuda")
    K = torch.empty((hkv, rows, D), dtype=torch.bfloat16, device="cuda")
    V = torch.empty((hkv, rows, D), dtype=torch.bfloat16, device="cuda")
    for kv in range(hkv):
        V[kv] = torch.randn((rows, D), generator=gen, device="cuda", dtype=torch.float32)
        k0 = _noise(gen, rows, D)
        k = k0.clone()
        for h in range(kv * g, (kv + 1) * g):
            q = _noise(gen, n, D)
            ch = PLANT_LO + h % 4
            if pats[h] == sa.SA_TRIANGULAR:  # four sinks, and a window over the query's own half-block and the one before
                k[:4, ch] = a
                q[:, ch] = a
                u = codes(nhalf)
                both = u.copy()
                both[1:] += u[:-1]
                k[:n, CODE_LO:] += a * torch.from_numpy(u).cuda()[idx_half]
                q[:, CODE_LO:] += a * torch.from_numpy(both).cuda()[idx_half]
            elif pats[h] == sa.SA_INTERVAL_SLASH:
                k[torch.from_numpy(host.choice(n - w, ncol, replace=False)).cuda(), ch] = a
                q[:, ch] = a
                for o in host.choice(n - w + 1, noff, replace=False):
                    o = int(o)
                    q[o:, :PLANT_LO] += gain * k0[: n - o, :PLANT_LO]
            elif pats[h] == sa.SA_BLOCK_CLUSTER:  # hot blocks, clustered on a few query bands where there are many
                ku, qu = np.zeros((nblk, D - CODE_LO), np.float32), np.zeros((nblk, D - CODE_LO), np.float32)
                r = host.randint(1, nblk, nhot if nhot == 32 else 4)
                r = r if nhot == 32 else np.repeat(r, nhot // 4)
                for R, u in zip(r, codes(nhot)):
                    ku[host.randint(0, R)] += u
                    qu[R] += u
                k[:n, CODE_LO:] += a * torch.from_numpy(ku).cuda()[idx_blk]
                q[:, CODE_LO:] += a * torch.from_numpy(qu).cuda()[idx_blk]
            Q[h] = q
        K[kv] = k
    return Q, K, V


def _score_reference(ses, Q, K):
    """Fills the session's score buffers with torch, in fp32: inputs of the calls that start from scores."""
    cfg = ses.cfg
    g, n, w, b = cfg.n_q_heads // cfg.n_kv_heads, cfg.seq_len, cfg.last_q, cfg.block
    nb = n // b
    hidden = torch.arange(n, device="cuda")[None, :] > torch.arange(n - w, n, device="cuda")[:, None]
    upper = torch.ones((nb, nb), dtype=torch.bool, device="cuda").triu(1)
    scale = 1.0 / math.sqrt(D)
    for h in range(cfg.n_q_heads):
        k = K[h // g, :n].float()
        p = (Q[h, n - w:].float() @ k.t()) * scale
        p = torch.softmax(p.masked_fill(hidden, float("-inf")), dim=1)
        ses.v[h] = p.sum(0)
        # row i's entry at offset o sits at o + w - 1 - i of the reversed row
        flat = torch.zeros((w, n + w), device="cuda")
        flat[:, :n] = p.flip(1)
        ses.s[h] = torch.as_strided(flat, (w, n), (n + w - 1, 1), w - 1).sum(0)
        m = (Q[h].float().view(nb, b, D).mean(1) @ k.view(nb, b, D).mean(1).t()) * scale
        ses.blk[h] = torch.softmax(m.masked_fill(upper, float("-inf")), dim=1).masked_fill(upper, 0.0)


class State:
    pass


def prepare(case, seed):
    s = State()
    s.kind = case["kind"]
    hq, hkv, n, block, w = case["hq"], case["hkv"], case["n"], case["block"], case["window"]
    # a generated token needs room behind the prompt's keys
    rows = n + max(64, case.get("generated", 0) + 1) if s.kind == "decode" else n
    s.Q, s.K, s.V = _inputs(case, seed, rows)
    more = {}
    if s.kind == "decode":
        more["kv_head_stride"] = rows * D
    if s.kind == "dense":
        nb = n // block
        more.update(local_blocks=nb, k_blocks=nb * (nb + 1) // 2)
    for k in ("block_select", "diagonal_select"):
        if case.get(k):
            more[k] = case[k]
    if case.get("lazy"):
        more["lazy_block_map"] = 1
    s.ses = sa.Session(hq, hkv, n, block, w, keep=case["keep"], **more)
    s.one_call = bool(case.get("one_call"))
    # -1, plain noise, is also the value that leaves the choice to the library
    s.override = _patterns(case) if case.get("override") else None
    if s.kind in ("layer", "dense"):
        s.O = torch.empty_like(s.Q)
    if s.kind == "dense":
        s.ses.estimate(s.Q, s.K)
        s.ses.build_index([sa.SA_TRIANGULAR] * hq)  # the band covers the sequence
    if s.kind in ("index", "decode", "search"):
        _score_reference(s.ses, s.Q, s.K)
    if s.kind == "decode":
        s.ses.build_index()
        s.pos = n + case["generated"] - 1
        s.q = torch.randn((hq, D), generator=torch.Generator(device="cuda").manual_seed(seed + 1), device="cuda").bfloat16()
        s.o = torch.empty_like(s.q)
        del s.Q
    if s.kind == "index":
        del s.Q, s.K, s.V
    if s.kind == "search":
        s.target = int(case["keep"] * n * (n + 1) / 2)
        s.eps = s.target // 200
    return s


def run(s):
    ses = s.ses
    if s.kind == "layer":
        if s.one_call:
            ses.estimate_and_index(s.Q, s.K, s.override)
        else:
            ses.estimate(s.Q, s.K)
            ses.build_index(s.override)
        ses.prefill(s.Q, s.K, s.V, s.O)
        return {"out": s.O, "pattern": ses.pattern}
    if s.kind == "dense":
        ses.prefill(s.Q, s.K, s.V, s.O)
        return s.O
    if s.kind == "estimate":
        ses.estimate(s.Q, s.K)
        return {"v": ses.v, "s": ses.s, "blk": ses.blk}
    if s.kind == "index":
        ses.build_index()
        return ses.index_tensors()
    if s.kind == "decode":
        ses.decode(s.q, s.K, s.V, s.pos, s.o)
        return s.o
    found = ses.search_patterns(s.Q, s.K, s.V, s.target, s.eps)
    return {"pattern": np.array([r["pattern"] for r in found]), "param": np.array([r["param"] for r in found]),
            "pairs": np.array([r["pairs"] for r in found]), "err": np.array([r["err"] for r in found])}


def _kept_pairs(case):
    """Kept (query, key) pairs of a layer, from its budgets and planted patterns."""
    n, b, keep = case["n"], case["block"], case["keep"]
    causal = n * (n + 1) / 2
    nb = n // b
    blocks = min(causal, max(keep * nb * (nb + 1) / 2, nb) * b * b)
    cols = 64 * max(1, round(keep * n / 256))
    slash = cols * n / 2 + max(1, round(keep * n / 128)) * n / 2 + n * b / 2
    return sum(min(causal, slash) if p == sa.SA_INTERVAL_SLASH else blocks for p in _patterns(case))


def work(case):
    hq, hkv, n, b, w, kind = case["hq"], case["hkv"], case["n"], case["block"], case["window"], case["kind"]
    nb = n // b
    q, kv = 2 * hq * n * D, 2 * hkv * n * D
    scores = 8 * hq * n + 4 * hq * nb * nb
    est = 2 * hq * w * n * D + hq * nb * (nb + 1) * D
    if kind == "estimate":
        return {"bytes": q + kv + scores, "flops": est}
    if kind == "index":
        cfg = sa.sa_default_budgets(sa.SaConfig(seq_len=n, block=b), case["keep"])
        return {"bytes": scores - 2 * hq * nb * (nb - 1) + 4 * hq * (cfg.k_vertical + cfg.k_slash + cfg.k_blocks + nb), "flops": 0}
    if kind == "decode":
        cfg = sa.sa_default_budgets(sa.SaConfig(seq_len=n, block=b), case["keep"])
        last = max(1, case["keep"] * nb) * b  # keys of the last row block's kept blocks
        keys = sum(cfg.k_vertical + cfg.k_slash + b if p == sa.SA_INTERVAL_SLASH else min(n, last) for p in _patterns(case))
        own = case["generated"]  # seen by every head of a group
        return {"bytes": 4 * D * (keys + hkv * own) + 4 * hq * D, "flops": 4 * D * (keys + hq * own)}
    if kind == "dense":
        return {"bytes": 2 * q + 2 * kv, "flops": 4 * D * hq * n * (n + 1) / 2}
    if kind == "search":  # per head the dense output and, of each candidate, the sparse one at the target
        pairs = n * (n + 1) / 2 * (1 + 3 * case["keep"])
        return {"bytes": q + 2 * kv, "flops": 4 * D * hq * pairs}
    return {"bytes": 2 * q + 2 * kv, "flops": est + 4 * D * _kept_pairs(case)}


def tolerance(case):
    if case["kind"] == "index":
        return "exact"
    if case["kind"] == "estimate":
        # fp32 sums of bf16 products; the block means enter the map's products as two bf16 parts each
        return {"rel": 1e-4}
    # bf16 outputs of softmax weights rounded to bf16; patterns and pair counts are whole numbers
    return {"rel": 1e-2, "differ": 0.0}
