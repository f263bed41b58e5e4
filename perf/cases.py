"""Timed cases of the cuckoo filter library: what a program has it do, through
its public entry points, over the range of sizes it is used at.

Kinds of case (a case is a dict of plain values):

  calls  one small round of calls on a resident filter: insert, query, delete.
  query  one batch of membership queries on a filled filter.
  build  empty a filter, insert a whole key set in one call, look some up.
  step   the update step of a filter kept at a high load: insert fresh keys,
         query, delete the oldest keys.
  set    one mixed (kind, filter, key) batch over a resident filter set.
  serve  a burst of requests through the serving loop, waited for.

Keys are uniform 64-bit integers (SplitMix64 streams of the case's seed), as
in the repository's own benchmark.  Loads stay where no insertion fails, so
every answer of a pass is determined by the inputs: outputs are flag bytes,
compared as whole numbers (there are no computed real numbers and so no
`exact`).  State changes by a closed cycle of key sets, so a pass can be
repeated any number of times.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_15486_amd as cf

NEG = 1 << 63           # counters from here on are never stored keys
RING = 1 << 40          # counters of the key sets that come and go
FILL = 1 << 24          # keys per call while a filter is filled in prepare()


# ------------------------------------------------------------------- cases

def _geom(buckets, b, f, load, hash="fmix64", evict="bfs", placement="xor"):
    return {"buckets": buckets, "b": b, "f": f, "load": load, "hash": hash, "evict": evict,
            "placement": placement}


def listed():
    return [
        # A service that checks a request's few keys against a small filter
        # as they come: what counts is the latency of single small calls.
        {"name": "calls_100", "kind": "calls", **_geom(1 << 18, 4, 16, 0.5), "n": 100},
        # The small end-to-end workload's queries: the table sits in cache.
        {"name": "query_2MiB", "kind": "query", **_geom(1 << 18, 4, 16, 0.9), "n": 1943718,
         "positive": 0.4855},
        # A table of the paper's throughput figure, an ordinary batch.
        {"name": "query_512MiB", "kind": "query", **_geom(1 << 24, 16, 16, 0.95), "n": 1 << 24,
         "positive": 0.5},
        # The benchmark's query launch: 4 GiB table, 2^26 keys, half stored.
        {"name": "query_4GiB", "kind": "query", **_geom(1 << 27, 16, 16, 0.945), "n": 1 << 26,
         "positive": 0.5},
        # Building the small workload's filter from its 943 718 keys.
        {"name": "build_2MiB", "kind": "build", **_geom(1 << 18, 4, 16, 0.9)},
        # Building a byte-per-key filter of short buckets: many evictions.
        {"name": "build_64MiB_f8", "kind": "build", **_geom(1 << 24, 4, 8, 0.9)},
        # Building a filter of 255 million keys in one call.
        {"name": "build_512MiB", "kind": "build", **_geom(1 << 24, 16, 16, 0.95)},
        # The benchmark's updates: 2^24 fresh keys in, 2^22 asked for, the
        # 2^24 oldest out, on the 4 GiB table between loads 0.942 and 0.95.
        {"name": "step_4GiB", "kind": "step", **_geom(1 << 27, 16, 16, 0.95), "n": 1 << 24,
         "queries": 1 << 22},
        # A deduplication step on a filter of an odd size: the offset
        # placement, 32-bit fingerprints, xxHash64, a ragged batch.
        {"name": "step_offset_f32", "kind": "step",
         **_geom(3 * (1 << 18) + 7, 8, 32, 0.9, "xxh64", "bfs", "offset"), "n": 300007,
         "queries": 1200013},
        # Mixed batches over 256 filters of 2^12..2^26 slots, one launch per
        # phase (what the tuner picks for it).
        {"name": "set_256_2e22", "kind": "set", "filters": 256, "lo": 12, "hi": 26, "f8": False,
         "n": 1 << 22, "fused": True},
        # A small mixed batch over filters of several classes in the
        # default launch shape.
        {"name": "set_24_20000", "kind": "set", "filters": 24, "lo": 14, "hi": 22, "f8": True,
         "n": 20000, "fused": False},
        # A burst of requests of 1..2^20 keys on 64 filters.
        {"name": "serve_64_burst", "kind": "serve", "filters": 64, "lo": 20, "hi": 26,
         "requests": 1024, "largest": 1 << 20},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_geom(rng, lo_slots, hi_slots, most_load):
    """A filter of lo..hi slots in any of the compiled geometries and options."""
    b = rng.choice([4, 8, 16, 16, 32])
    f = rng.choice([8, 16, 16, 32])
    placement = rng.choice(["xor", "xor", "offset"])
    slots = _log(rng, lo_slots, hi_slots)
    buckets = max(64, int(slots / b))
    if placement == "xor":
        buckets = 1 << max(6, round(math.log2(buckets)))
        while buckets * b > hi_slots:
            buckets >>= 1
    load = min(most_load, {4: 0.85, 8: 0.9, 16: 0.95, 32: 0.95}[b])
    return _geom(buckets, b, f, round(rng.uniform(0.5, load), 3),
                 rng.choice(["fmix64", "fmix64", "xxh64"]),
                 rng.choice(["bfs", "bfs", "bfs", "dfs"]), placement)


def draw(rng):
    kind = rng.choice(["calls", "query", "query", "query", "build", "build", "step", "step",
                       "set", "serve"])
    if kind == "calls":
        return {"kind": kind, **_draw_geom(rng, 1 << 16, 1 << 26, 0.7), "n": int(_log(rng, 16, 4096))}
    if kind == "query":
        g = _draw_geom(rng, 1 << 18, 1 << 30, 0.95)
        return {"kind": kind, **g, "n": int(_log(rng, 1 << 12, 1 << 25)),
                "positive": round(rng.choice([0.02, 0.98, rng.uniform(0.02, 0.98)]), 3)}
    if kind == "build":
        return {"kind": kind, **_draw_geom(rng, 1 << 18, 1 << 27, 0.95)}
    if kind == "step":
        g = _draw_geom(rng, 1 << 20, 1 << 29, 0.93)
        most = min(1 << 23, g["buckets"] * g["b"] // 32)
        n = int(_log(rng, 1 << 10, most))
        return {"kind": kind, **g, "n": n, "queries": rng.choice([n // 4, n, 3 * n])}
    if kind == "set":
        f8 = rng.random() < 0.5
        return {"kind": kind, "filters": rng.choice([3, 17, 64, 200]), "lo": rng.choice([12, 14]),
                "hi": rng.choice([18, 20, 22]), "f8": f8, "n": int(_log(rng, 1 << 10, 1 << 20)),
                "fused": (not f8) and rng.random() < 0.5}
    return {"kind": kind, "filters": rng.choice([8, 32, 64]), "lo": 18, "hi": rng.choice([20, 24]),
            "requests": int(_log(rng, 64, 1024)), "largest": int(_log(rng, 1 << 8, 1 << 18))}


# ----------------------------------------------------------------- prepare

_HASH = {"fmix64": cf.CF_HASH_FMIX64, "xxh64": cf.CF_HASH_XXH64}
_EVICT = {"bfs": cf.CF_EVICT_BFS, "dfs": cf.CF_EVICT_DFS}
_PLACE = {"xor": cf.CF_PLACE_XOR, "offset": cf.CF_PLACE_OFFSET}


def _filter(case, seed):
    return cf.CuckooFilter(case["buckets"], case["b"], case["f"], hash=_HASH[case["hash"]],
                           evict=_EVICT[case["evict"]],
                           max_evict=128 if case["evict"] == "bfs" else 500, seed=seed,
                           placement=_PLACE[case["placement"]])


def _keys(seed, start, n):
    k = torch.empty(n, dtype=torch.int64, device="cuda")
    cf.cf_keygen(k, seed, start)
    return k


def _keys_at(seed, counters):
    k = torch.empty(counters.numel(), dtype=torch.int64, device="cuda")
    cf.cf_keygen_at(k, counters, seed)
    return k


def _flags(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def _fill(flt, seed, n):
    for lo in range(0, n, FILL):
        flt.insert(_keys(seed, lo, min(FILL, n - lo)))


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _probe_keys(seed, stored, n, positive, gen):
    """n keys in random order, a share `positive` of them stored ones."""
    hit = torch.rand(n, generator=gen, device="cuda") < positive
    at = torch.randint(0, max(1, stored), (n,), generator=gen, device="cuda")
    neg = torch.arange(n, device="cuda") + (NEG - (1 << 64))
    return _keys_at(seed, torch.where(hit, at, neg))


def _prepare_calls(case, seed):
    flt = _filter(case, seed)
    stored = int(case["load"] * flt.capacity)
    _fill(flt, seed, stored)
    n = case["n"]
    new = _keys(seed, RING, n)
    flt.reserve(FILL)
    return {"flt": flt, "new": new,
            "ask": torch.cat([new, _probe_keys(seed, stored, n, 0.5, _gen(seed))]),
            "ok_in": _flags(n), "found": _flags(2 * n), "ok_out": _flags(n)}


def _prepare_query(case, seed):
    flt = _filter(case, seed)
    stored = int(case["load"] * flt.capacity)
    _fill(flt, seed, stored)
    n = case["n"]
    return {"flt": flt, "keys": _probe_keys(seed, stored, n, case["positive"], _gen(seed)),
            "found": _flags(n)}


def _prepare_build(case, seed):
    flt = _filter(case, seed)
    n = int(case["load"] * flt.capacity)
    flt.reserve(n)
    return {"flt": flt, "keys": _keys(seed, 0, n), "ok": _flags(n),
            "ask": _probe_keys(seed, n, max(1, n // 16), 0.5, _gen(seed)),
            "found": _flags(max(1, n // 16))}


SETS, KEPT = 8, 7       # key sets of a step's ring, and how many are stored


def _prepare_step(case, seed):
    flt = _filter(case, seed)
    n, q = case["n"], case["queries"]
    stored = int(case["load"] * flt.capacity) - (KEPT + 1) * n
    _fill(flt, seed, stored)
    sets = [_keys(seed, RING + k * n, n) for k in range(SETS)]
    flt.reserve(max(n, min(FILL, stored)))
    for k in range(KEPT):
        flt.insert(sets[k])
    gen = _gen(seed)
    return {"flt": flt, "sets": sets, "pass": 0,
            "ask": _probe_keys(seed, stored, q, 0.5, gen),
            "ok_in": _flags(n), "ok_out": _flags(n), "found": _flags(q)}


def _set_params(case, seed):
    """Filters of 2^lo..2^hi slots with 8 or 16 slots per bucket."""
    r = np.random.default_rng(seed)
    params, slots = [], []
    for i in range(case["filters"]):
        b = int(r.choice([8, 16]))
        f = int(r.choice([8, 16])) if case.get("f8") else 16
        s = 1 << int(r.integers(case["lo"], case["hi"] + 1))
        params.append(cf.make_params(s // b, b, f, seed=seed + i))
        slots.append(s)
    return params, np.array(slots, dtype=np.int64), r


def _prepare_set(case, seed):
    """Batches of 60% queries, 20% deletes and 20% inserts; the inserts of one
    batch are the deletes of a later one."""
    params, slots, r = _set_params(case, seed)
    n = case["n"]
    st = cf.CuckooFilterSet(params, max(n, 1 << 22))
    if case["fused"]:
        st.set_shape(fused=1)
    stored = (slots * r.uniform(0.5, 0.85, slots.size)).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(stored)])[:-1]
    for f in range(slots.size):
        for lo in range(0, int(stored[f]), st.max_batch):
            st.apply(f, cf.CF_OP_INSERT,
                     _keys(seed, int(off[f]) + lo, min(st.max_batch, int(stored[f]) - lo)))
    gen = _gen(seed)
    share = torch.from_numpy(slots / slots.sum()).cuda().cumsum(0)

    def pick(k):
        u = torch.rand(k, generator=gen, device="cuda", dtype=torch.float64)
        return torch.searchsorted(share, u).clamp_(max=slots.size - 1)

    d_off, d_stored = torch.from_numpy(off).cuda(), torch.from_numpy(stored).cuda()
    n_up = max(1, n // 5)
    n_q = max(1, n - 2 * n_up)
    sets = [(pick(n_up), _keys(seed, RING + k * n_up, n_up)) for k in range(4)]
    for k in range(2):
        ops = torch.full((n_up,), cf.CF_OP_INSERT, dtype=torch.uint8, device="cuda")
        st.execute(ops, sets[k][0].to(torch.int32), sets[k][1])
    batches = []
    for p in range(4):
        qf = pick(n_q)
        u = torch.rand(n_q, generator=gen, device="cuda", dtype=torch.float64)
        at = d_off[qf] + (u * d_stored[qf]).to(torch.int64)
        neg = torch.arange(n_q, device="cuda") + (NEG - (1 << 64)) + p * n_q
        hit = torch.rand(n_q, generator=gen, device="cuda") < 0.5
        fids = torch.cat([qf, sets[p][0], sets[(p + 2) % 4][0]])
        keys = torch.cat([_keys_at(seed, torch.where(hit, at, neg)), sets[p][1],
                          sets[(p + 2) % 4][1]])
        ops = torch.cat([torch.full((n_q,), cf.CF_OP_QUERY, dtype=torch.uint8, device="cuda"),
                         torch.full((n_up,), cf.CF_OP_DELETE, dtype=torch.uint8, device="cuda"),
                         torch.full((n_up,), cf.CF_OP_INSERT, dtype=torch.uint8, device="cuda")])
        order = torch.randperm(ops.numel(), generator=gen, device="cuda")
        batches.append((ops[order].contiguous(), fids[order].to(torch.int32).contiguous(),
                        keys[order].contiguous()))
    return {"set": st, "batches": batches, "pass": 0,
            "results": [_flags(b[0].numel()) for b in batches]}


def _prepare_serve(case, seed):
    """70% queries; the rest insert a key set that a later request deletes.
    The filters and the trace's sizes belong to the case, the keys to the seed."""
    params, slots, r = _set_params(case, case["requests"])
    largest = case["largest"]
    srv = cf.CuckooServer(params, max_batch=1 << 22, max_requests=4096, depth=8)
    stored = (slots * r.uniform(0.5, 0.75, slots.size)).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(stored)])[:-1]
    for f in range(slots.size):
        for lo in range(0, int(stored[f]), 1 << 22):
            srv.set.apply(f, cf.CF_OP_INSERT,
                          _keys(seed, int(off[f]) + lo, min(1 << 22, int(stored[f]) - lo)))
    count = case["requests"]
    room = (slots * 0.1).astype(np.int64)     # slots that updates may take at once
    where = np.sort(r.random(count))
    reqs, ring = [], RING
    while len(reqs) < count:
        n = max(1, min(largest, int(math.exp(r.uniform(0, math.log(largest))))))
        fit = np.flatnonzero(slots >= 8 * n)
        if fit.size == 0:
            continue
        f = int(r.choice(fit, p=slots[fit] / slots[fit].sum()))
        a = float(where[len(reqs)])
        if r.random() < 0.7 or len(reqs) + 2 > count or n > room[f]:
            reqs.append((a, f, cf.CF_OP_QUERY, n, 0))
        else:
            room[f] -= n
            reqs.append((a, f, cf.CF_OP_INSERT, n, ring))
            reqs.append((float(r.uniform(a, 1.0)), f, cf.CF_OP_DELETE, n, ring))
            ring += n
    reqs.sort(key=lambda q: q[0])
    ns = np.array([q[3] for q in reqs], dtype=np.uint64)
    key_off = np.concatenate([[0], np.cumsum(ns)])[:-1].astype(np.uint64)
    total = int(ns.sum())
    gen = _gen(seed)
    keys = torch.empty(total, dtype=torch.int64, device="cuda")
    neg = NEG - (1 << 64)
    for q, ko in zip(reqs, key_off):
        n, f, ko = q[3], q[1], int(ko)
        if q[2] == cf.CF_OP_QUERY:
            hit = torch.rand(n, generator=gen, device="cuda") < 0.5
            at = torch.randint(0, int(stored[f]), (n,), generator=gen, device="cuda") + int(off[f])
            c = torch.where(hit, at, torch.arange(n, device="cuda") + (neg + ko))
            cf.cf_keygen_at(keys[ko:ko + n], c, seed)
        else:
            cf.cf_keygen(keys[ko:ko + n], seed, q[4])
    torch.cuda.synchronize()
    return {"srv": srv, "arrival": np.zeros(count, dtype=np.uint64),
            "fids": np.array([q[1] for q in reqs], dtype=np.uint32),
            "ops": np.array([q[2] for q in reqs], dtype=np.uint32), "key_off": key_off, "n": ns,
            "keys": keys, "results": _flags(total)}


_PREPARE = {"calls": _prepare_calls, "query": _prepare_query, "build": _prepare_build,
            "step": _prepare_step, "set": _prepare_set, "serve": _prepare_serve}


def prepare(case, seed):
    state = _PREPARE[case["kind"]](case, (seed * 1000003 + 12345) & (2**62 - 1))
    state["kind"] = case["kind"]
    return state


# --------------------------------------------------------------------- run

def run(state):
    kind = state["kind"]
    if kind == "query":
        return state["flt"].query(state["keys"], state["found"])
    if kind == "calls":
        flt = state["flt"]
        return [flt.insert(state["new"], state["ok_in"]), flt.query(state["ask"], state["found"]),
                flt.delete(state["new"], state["ok_out"])]
    if kind == "build":
        flt = state["flt"]
        flt.reset()
        return [flt.insert(state["keys"], state["ok"]), flt.query(state["ask"], state["found"])]
    if kind == "step":
        flt, p = state["flt"], state["pass"]
        state["pass"] = p + 1
        return [flt.insert(state["sets"][(p + KEPT) % SETS], state["ok_in"]),
                flt.query(state["ask"], state["found"]),
                flt.delete(state["sets"][p % SETS], state["ok_out"])]
    if kind == "set":
        p = state["pass"] % 4
        state["pass"] += 1
        ops, fids, keys = state["batches"][p]
        return state["set"].execute(ops, fids, keys, state["results"][p])
    srv = state["srv"]
    srv.replay(state["arrival"], state["fids"], state["ops"], state["key_off"], state["n"],
               state["keys"], state["results"])
    srv.drain()
    return state["results"]


# -------------------------------------------------------------------- work

def _probe_bytes(n, per_key, bucket, table):
    """Bucket bytes that n keys read, a table at most once."""
    return min(n * per_key * bucket, table)


def work(case):
    kind = case["kind"]
    if kind in ("calls", "query", "build", "step"):
        bucket = case["b"] * case["f"] / 8
        table = case["buckets"] * bucket
        up = lambda n: n * 9 + 2 * _probe_bytes(n, 1, bucket, table)  # noqa: E731
        ask = lambda n, pos: n * 9 + _probe_bytes(n, 2 - pos, bucket, table)  # noqa: E731
        n = case.get("n", 0)
        if kind == "query":
            total = ask(n, case["positive"])
        elif kind == "calls":
            total = 2 * up(n) + ask(2 * n, 0.75)
        elif kind == "build":
            n = int(case["load"] * case["buckets"] * case["b"])
            total = n * 9 + table + ask(max(1, n // 16), 0.5)
        else:
            total = 2 * up(n) + ask(case["queries"], 0.5)
        return {"bytes": total, "flops": 0}
    # 16-bit slots, 12 slots per bucket on average: 24 bytes a bucket
    if kind == "set":
        n = case["n"]
        return {"bytes": n * 14 + 0.6 * n * 1.5 * 24 + 0.4 * n * 2 * 24, "flops": 0}
    mean = (case["largest"] - 1) / max(1e-9, math.log(case["largest"]))
    n = case["requests"] * mean
    return {"bytes": n * 9 + 0.7 * n * 1.5 * 24 + 0.3 * n * 2 * 24, "flops": 0}
