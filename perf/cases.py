"""Performance cases of the cached mixed-precision EmbeddingBag step.

A case is one workload shape and one way of calling the library on it:

  step     forward, then backward_update: one training step;
  forward  the forward alone, with the handle's workspace (evaluation, serving);
  noalloc  forward_noalloc into a buffer of the caller's (serving under graph capture).

`prepare` makes what a training or serving program holds before such a call: the handle
with a warm cache, a few batches of indices and offsets, and output gradients, on the
GPU.  A model of at most IMPORT_CODES codes is loaded from generated arrays, as from a
checkpoint; a larger one is initialised by the library and trained for a few steps on
other batches.  `run` takes the batches in turn, so that a repeated pass does not find
its own rows in the cache more often than a training program would.

The results of the library are reproducible bit for bit (the order of every sum is part
of its interface), so every case is compared exactly.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2010_11305_amd import configs
from paper_2010_11305_amd.emb_cache import EmbCache

BATCHES = 3        # index batches a state holds
WARM_STEPS = 3     # training steps of a model too large to load
IMPORT_CODES = 1 << 26
LR, EPS, SEED = 0.01, 1e-8, 2


def _case(name, mode, tables, rows, dim, bits, frac, assoc, policy, batch, pool, mean, zipf, sb16=False, decay=0,
          sr=False, adagrad=False, host=False):
    """`rows` 0: the 26 tables of Table 1 of the paper.  Bags: `pool` "fixed" (mean lookups
    each), "poisson" (that mean) or "uniform" (1 .. 2*mean - 1)."""
    c = dict(mode=mode, tables=tables, rows=rows, dim=dim, bits=bits, sb16=sb16, frac=frac, assoc=assoc,
             policy=policy, decay=decay, sr=sr, adagrad=adagrad, batch=batch, pool=pool, mean=mean, zipf=zipf,
             host=host)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest training step: one small table, 128 bags of 1..4 lookups (the `tiny`
        # workload); what an online learner or a unit of a pipeline test calls
        _case("tiny_step", "step", 1, 1000, 16, 8, 0.05, 4, "lru", 128, "uniform", 2.5, 1.05),
        # ranking requests served one small batch at a time on the 26 Criteo-Kaggle-shaped tables
        _case("kaggle_serve", "noalloc", 26, 0, 16, 8, 0.05, 32, "lru", 256, "fixed", 1, 1.1),
        # training on those tables, batch 2048, INT8, 5% cache, LRU, SGD (the `kaggle_int8` workload)
        _case("kaggle_int8_step", "step", 26, 0, 16, 8, 0.05, 32, "lru", 2048, "fixed", 1, 1.1),
        # the same tables in INT4 with FP16 (s, b), 1% cache, LFU with decay, stochastic
        # rounding, Adagrad, batch 8192 (the `kaggle_int4` workload)
        _case("kaggle_int4_step", "step", 26, 0, 16, 4, 0.01, 32, "lfu", 8192, "fixed", 1, 1.1, sb16=True, decay=10,
              sr=True, adagrad=True),
        # the hit-rate study's stream: one table of 1M rows, direct-mapped LFU, one lookup per sample
        _case("hitrate_step", "step", 1, 1_000_000, 16, 8, 0.05, 1, "lfu", 16384, "fixed", 1, 1.05),
        # evaluation of a multi-hot model: 12 tables of 83,333 rows, INT4, 8 ways, ragged bags
        _case("multihot_eval", "forward", 12, 83_333, 64, 4, 0.05, 8, "lru", 1000, "poisson", 20, 1.1, sb16=True),
        # training of a mid-sized ranker: 10 tables of 100,003 rows, INT8, odd batch, ragged bags
        _case("ranker_step", "step", 10, 100_003, 64, 8, 0.05, 16, "lru", 4099, "poisson", 12, 1.1),
        # serving the 100-table industrial shape (500k rows each here) at batch 512
        _case("industrial_serve", "forward", 100, 500_000, 128, 4, 0.01, 16, "lru", 512, "poisson", 30, 1.2, sb16=True,
              adagrad=True, sr=True),
        # ten tables of the industrial shape stored in FP16, the paper's industrial precision
        _case("fp16_step", "step", 10, 5_000_000, 128, 16, 0.01, 16, "lru", 16384, "poisson", 30, 1.2, adagrad=True),
        # the low-precision table in pinned host memory (the paper's Fig. 9), 2% cache
        _case("host_table_step", "step", 4, 250_000, 128, 16, 0.02, 16, "lru", 4096, "poisson", 30, 1.2, adagrad=True,
              host=True),
        # one table of 200M rows of 256 columns, INT8, 64 lookups per bag (the `stress` workload)
        _case("stress_step", "step", 1, 200_000_000, 256, 8, 0.01, 32, "lru", 65536, "fixed", 64, 1.05, sr=True),
        # the full industrial training step: 100 tables of 5M rows (the benchmark's workload)
        _case("industrial_step", "step", 100, 5_000_000, 128, 4, 0.01, 16, "lru", 16384, "poisson", 30, 1.2, sb16=True,
              sr=True, adagrad=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another shape of the same ranges: calls from a hundred to ten million lookups, 1 to
    100 tables of a thousand to five million rows or those of Table 1, every row width,
    precision, policy, rounding and optimizer."""
    mode = rng.choice(["step", "step", "step", "forward", "noalloc"])
    policy = rng.choice(["lru", "lru", "lfu"])
    bits = rng.choice([4, 8, 8, 4, 16, 2])
    common = dict(policy=policy, bits=bits, sb16=bits != 16 and rng.random() < 0.5,
                  decay=rng.choice([0, 10]) if policy == "lfu" else 0, sr=rng.random() < 0.5,
                  adagrad=rng.random() < 0.5)
    if rng.random() < 0.3:
        return _case(None, mode, 26, 0, rng.choice([16, 16, 32]), frac=rng.choice([0.01, 0.05]),
                     assoc=rng.choice([16, 32]), batch=_log_uniform(rng, 32, 16384), pool="fixed", mean=1,
                     zipf=round(rng.uniform(1.05, 1.2), 2), **common)
    host = mode == "step" and rng.random() < 0.08
    dim = rng.choice([16, 32, 64, 128, 256])
    tables = _log_uniform(rng, 1, 8 if host else 100)
    rows = _log_uniform(rng, 1000, min(5_000_000, (200_000_000 if host else 20_000_000_000) // (2 * dim * tables)))
    mean = rng.choice([1, 2, 4, 10, 20, 30, 50])
    most = min(10_000_000 // (tables * mean), 200_000_000 // (tables * dim), 500_000 // (mean * tables) if host else 10**9)
    batch = _log_uniform(rng, 16, max(32, min(65536, most)))
    return _case(None, mode, tables, rows, dim, frac=rng.choice([0.01, 0.02, 0.05]), assoc=rng.choice([1, 4, 8, 16, 32, 64]),
                 batch=batch, pool="fixed" if mean == 1 else rng.choice(["fixed", "poisson", "uniform"]), mean=mean,
                 zipf=round(rng.uniform(1.05, 1.25), 2), host=host, **common)


# ---- shapes ---------------------------------------------------------------------------------
def _rows(case):
    return list(configs.TABLE1_ROWS) if case["rows"] == 0 else [case["rows"]] * case["tables"]


def _config(case):
    return dict(rows=_rows(case), dim=case["dim"], bits=case["bits"], sb_fp16=case["sb16"],
                cache_fraction=case["frac"], assoc=case["assoc"], policy=case["policy"],
                lfu_decay_interval=case["decay"], rounding="stochastic" if case["sr"] else "nearest",
                optimizer="adagrad" if case["adagrad"] else "sgd", lr=LR, eps=EPS, seed=SEED, batch=case["batch"])


def _sets(case, n):
    return max(1, int(case["frac"] * n) // case["assoc"])


def _loaded(case):
    return sum(_rows(case)) * case["dim"] <= IMPORT_CODES


# ---- inputs ---------------------------------------------------------------------------------
def _generator(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1_000_003 + what) % (1 << 62))
    return g


def _bijection(seed, n, t):
    """(a, c): the row of popularity rank k (from 0) is (a*k + c) mod n."""
    r = np.random.default_rng([seed, t])
    while True:
        a = int(r.integers(1, max(n, 2)))
        if math.gcd(a, n) == 1:
            return a, int(r.integers(0, n))


def _batch(case, seed, what):
    """(indices, offsets): Zipf ranks by inversion of the integral of x**-zipf, scattered
    over the rows by a bijection; table-major bags."""
    g = _generator(seed, what)
    rows, B, mean = _rows(case), case["batch"], case["mean"]
    T = len(rows)
    if case["pool"] == "fixed":
        lengths = torch.full((T * B,), int(mean), dtype=torch.int64, device="cuda")
    elif case["pool"] == "poisson":
        lengths = torch.poisson(torch.full((T * B,), float(mean), device="cuda"), generator=g).to(torch.int64)
    else:
        lengths = torch.randint(1, int(2 * mean), (T * B,), generator=g, device="cuda")
    offsets = torch.zeros(T * B + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lengths, 0, out=offsets[1:])
    first = offsets[::B].tolist()
    indices = torch.empty(max(first[-1], 1), dtype=torch.int32, device="cuda")[:first[-1]]
    e = 1.0 - case["zipf"]
    for t, n in enumerate(rows):
        u = torch.rand(first[t + 1] - first[t], generator=g, device="cuda", dtype=torch.float64)
        lo, hi = 0.5 ** e, (n + 0.5) ** e
        rank = (lo + u * (hi - lo)).pow_(1.0 / e).round_().clamp_(1, n).to(torch.int64) - 1
        a, c = _bijection(seed, n, t)
        indices[first[t]:first[t + 1]] = rank.mul_(a).add_(c).remainder_(n)
    return indices, offsets.to(torch.int32)


def _grad(case, seed, k):
    shape = (case["batch"], len(_rows(case)), case["dim"])
    return torch.randn(shape, generator=_generator(seed, 500 + k), device="cuda").mul_(0.01)


def _model_table(case, seed, t):
    """Table t of a stored model: low-precision rows, and a cache that holds the most popular
    rows of every set, its stamps from the last steps."""
    g = _generator(seed, 1000 + t)
    n, d, A = _rows(case)[t], case["dim"], case["assoc"]
    m = {"scale": torch.zeros(n, device="cuda"), "bias": torch.zeros(n, device="cuda")}
    if case["bits"] == 16:
        half = (torch.rand((n, d), generator=g, device="cuda") * 0.1 - 0.05).half()
        m["codes"], low = half, half.double()
    else:
        K = 2 ** case["bits"] - 1
        m["codes"] = torch.randint(0, K + 1, (n, d), generator=g, device="cuda", dtype=torch.uint8)
        m["scale"] = (torch.rand(n, generator=g, device="cuda") + 0.5) * (0.1 / K)
        m["bias"] = -0.05 - 0.01 * torch.rand(n, generator=g, device="cuda")
        if case["sb16"]:
            m["scale"], m["bias"] = m["scale"].half().float(), m["bias"].half().float()
        low = m["codes"].double() * m["scale"].double()[:, None] + m["bias"].double()[:, None]
    m["G"] = torch.rand(n, generator=g, device="cuda") * 1e-3
    m["cnt"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    S = _sets(case, n)
    a, c = _bijection(seed, n, t)
    ranked = torch.arange(n, device="cuda").mul_(a).add_(c).remainder_(n)
    key, order = torch.sort(ranked % S, stable=True)
    place = torch.arange(n, device="cuda") - torch.searchsorted(key, key)
    keep = place < A
    tag = torch.full((S * A,), -1, dtype=torch.int64, device="cuda")
    tag[key[keep] * A + place[keep]] = ranked[order][keep]
    m["tag"] = tag.to(torch.int32)
    noise = torch.randn((S * A, d), generator=g, device="cuda").double() * 1e-3
    m["crow"] = torch.where((tag >= 0)[:, None], low[tag.clamp(min=0)] + noise, torch.zeros_like(noise)).float()
    stamp = torch.randint(0, 8, (S * A,), generator=g, device="cuda", dtype=torch.int32)
    m["ts"] = torch.where(tag >= 0, stamp, torch.full_like(stamp, -1))
    if case["policy"] == "lfu":
        m["cnt"][ranked] = (2000 / torch.arange(1, n + 1, device="cuda").float()).to(torch.int32)
    return m, low


def prepare(case, seed):
    cfg = _config(case)
    batches = [_batch(case, seed, k) for k in range(BATCHES)]
    grads = [_grad(case, seed, k) for k in range(2)] if case["mode"] == "step" else []
    loaded = _loaded(case)
    warm = [] if loaded else [_batch(case, seed, 100 + k) for k in range(WARM_STEPS)]
    most = max(max(idx.numel() for idx, _ in batches + warm), 1)
    emb = EmbCache(cfg, max_indices=most, table="host" if case["host"] else "device")
    if loaded:
        for t in range(len(cfg["rows"])):
            m, _ = _model_table(case, seed, t)
            codes = m["codes"].view(torch.int16).cpu().numpy().view(np.uint16) if case["bits"] == 16 \
                else m["codes"].cpu().numpy()
            emb.import_rows(t, 0, codes, m["scale"].cpu().numpy(), m["bias"].cpu().numpy(), m["cnt"].cpu().numpy(),
                            m["G"].cpu().numpy())
            emb.import_cache(t, m["crow"].cpu().numpy(), m["tag"].cpu().numpy(), m["ts"].cpu().numpy())
        emb.step = 8
    else:
        emb.init_uniform(-0.05, 0.05, 1 + seed)
        g = grads[0] if grads else _grad(case, seed, 0)
        for idx, off in warm:
            emb.forward(idx, off, case["batch"])
            emb.backward_update(idx, off, case["batch"], g)
    state = {"emb": emb, "batches": batches, "grads": grads, "pass": 0, "mode": case["mode"], "B": case["batch"]}
    if case["mode"] == "noalloc":
        state["out"] = torch.empty((case["batch"], len(cfg["rows"]), case["dim"]), device="cuda")
    elif case["mode"] == "step":
        # the updated weights: the FP32 cache rows, and the records of the low-precision table
        s = emb.sizes
        state["cache"] = emb.state[:s.total_slots * case["dim"] * 4].view(torch.float32)
        table = emb.table if case["host"] else emb.state[s.state_bytes - s.table_bytes:s.state_bytes]
        records = s.total_rows * s.row_bytes
        state["table"] = table[:records].view(torch.int64 if records % 8 == 0 else torch.int32)
    torch.cuda.synchronize()
    return state


# ---- one pass -------------------------------------------------------------------------------
def run(state):
    k = state["pass"]
    state["pass"] = k + 1
    emb, B = state["emb"], state["B"]
    idx, off = state["batches"][k % BATCHES]
    if state["mode"] == "noalloc":
        return {"pooled": emb.forward_noalloc(idx, off, B, state["out"])}
    pooled = emb.forward(idx, off, B)
    if state["mode"] == "forward":
        return {"pooled": pooled}
    emb.backward_update(idx, off, B, state["grads"][k % 2])
    return {"pooled": pooled, "cache": state["cache"], "table": state["table"]}


# ---- what a pass cannot do without ----------------------------------------------------------
def _expected_unique(n, lookups, zipf, slots):
    """Expected distinct rows among `lookups` Zipf draws of n rows, and those of them among
    the `slots` most popular rows."""
    edges = np.unique(np.concatenate([np.arange(1, min(n, 4096) + 1), np.geomspace(1, n, 4000).astype(np.int64),
                                      [min(max(slots, 1), n), n]])).astype(np.float64)
    e = 1.0 - zipf
    mass = ((edges[:-1] + 0.5) ** e - (edges[1:] + 0.5) ** e) / (0.5 ** e - (n + 0.5) ** e) if n > 1 else np.zeros(0)
    count = np.diff(edges)
    head = (0.5 ** e - 1.5 ** e) / (0.5 ** e - (n + 0.5) ** e)
    seen = np.concatenate([[-math.expm1(-lookups * head)], -count * np.expm1(-lookups * mass / np.maximum(count, 1))])
    return float(seen.sum()), float(seen[edges <= slots].sum())


def work(case):
    rows, d, B = _rows(case), case["dim"], case["batch"]
    T = len(rows)
    L = case["mean"] * B * T
    record = d * case["bits"] // 8 + (0 if case["bits"] == 16 else 4 if case["sb16"] else 8)
    U = H = 0.0
    known = {}
    for n in rows:
        if n not in known:
            known[n] = _expected_unique(n, case["mean"] * B, case["zipf"], _sets(case, n) * case["assoc"])
        U, H = U + known[n][0], H + known[n][1]
    fetch = 4 * d * H + record * (U - H)                   # every row once, from the cache or the table
    nbytes = 4 * L + 4 * (T * B + 1) + 4 * case["assoc"] * min(U, sum(_sets(case, n) for n in rows)) + fetch + 4 * d * T * B
    flops = 3 * d * L                                       # q*s + b, then the sum
    if case["mode"] == "step":
        nbytes += 4 * L + 4 * d * T * B + 2 * fetch + (8 * U if case["adagrad"] else 0) + 4 * U
        flops += d * L + 4 * d * U
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    return "exact"


# ---- the same in 64 bits --------------------------------------------------------------------
def exact(case, seed):
    """The first pass on a loaded model, in float64.  The cache after a step is given for LRU
    with two or more ways (every missed row, in row order, takes the oldest way of its set
    that was not hit); the table's records are codes, not numbers."""
    if not _loaded(case):
        return None
    rows, d, A, B = _rows(case), case["dim"], case["assoc"], case["batch"]
    idx, off = _batch(case, seed, 0)
    step = case["mode"] == "step"
    grad = _grad(case, seed, 0).double() if step else None
    pooled = torch.zeros((B, len(rows), d), dtype=torch.float64, device="cuda")
    caches = []
    first = off[::B].tolist()
    for t, n in enumerate(rows):
        m, low = _model_table(case, seed, t)
        eff = low.clone()
        tag = m["tag"].long()
        held = tag >= 0
        eff[tag[held]] = m["crow"].double()[held]
        i = idx[first[t]:first[t + 1]].long()
        lengths = torch.diff(off[t * B:(t + 1) * B + 1].long())
        bag = torch.repeat_interleave(torch.arange(B, device="cuda"), lengths)
        for a in range(0, i.numel(), 1 << 20):
            pooled[:, t].index_add_(0, bag[a:a + (1 << 20)], eff[i[a:a + (1 << 20)]])
        if not step or case["policy"] != "lru" or A == 1:
            continue
        g = torch.zeros((n, d), dtype=torch.float64, device="cuda")
        for a in range(0, i.numel(), 1 << 20):
            g.index_add_(0, i[a:a + (1 << 20)], grad[bag[a:a + (1 << 20)], t])
        lr = torch.full((n,), float(np.float32(LR)), dtype=torch.float64, device="cuda")
        if case["adagrad"]:
            lr = lr / ((m["G"].double() + g.square().mean(1)).sqrt() + EPS)
        new = eff - lr[:, None] * g
        touched = torch.zeros(n, dtype=torch.bool, device="cuda")
        touched[i] = True
        S = _sets(case, n)
        hit = held & touched[tag.clamp(min=0)]
        cache = m["crow"].double()
        cache[hit] = new[tag[hit]]
        resident = torch.zeros(n, dtype=torch.bool, device="cuda")
        resident[tag[held]] = True
        missed = torch.nonzero(touched & ~resident).flatten()
        key, order = torch.sort(missed % S, stable=True)
        place = torch.arange(key.numel(), device="cuda") - torch.searchsorted(key, key)
        age = torch.where(hit, torch.full_like(tag, 1 << 20), m["ts"].long()).view(S, A)
        ways = torch.sort(age, dim=1, stable=True).indices
        enter = place < (A - hit.view(S, A).sum(1))[key]
        slot = key[enter] * A + ways[key[enter], place[enter]]
        cache[slot] = new[missed[order][enter]]
        caches.append(cache.flatten())
    if not step:
        return {"pooled": pooled}
    return {"pooled": pooled, "cache": torch.cat(caches) if caches else None, "table": None}
