"""Workloads by which the speed of the hash tables is followed.

Each case is one call, or one short chain of calls, that a program using the
tables makes: a lookup batch on a resident table, a table rebuilt from new
pairs and then queried (bulk build and probe), many tables built and queried
as one batch, many small lookup requests answered by one coalesced launch.
Sizes are those of the benchmark's workloads (headline, schemes, latency,
batched, serving) and of the GPU tests, scaled so that a pass stays within
some milliseconds; inputs are uniform unique keys with random values, the
benchmark's distribution, made on the GPU.

Fields of a case: "kind" (lookup, rebuild, batch, requests), "scheme" (bcht,
bcht64, bp2ht, iht), "n" pairs, "q" queries, "positive" share of queries that
are stored keys, "lf" load factor; a batch has "tables" with sizes
log-uniform in [2^lo, 2^hi]; requests are "count" lookups of log-uniform sizes
in [2^qlo, 2^qhi] on "tables" resident tables.
"""
import math
import random

import torch

import paper_2108_07232_amd as bht

M32 = 0xFFFFFFFF


def listed():
    return [
        # an online lookup of a few hundred keys: launch and latency
        {"name": "lookup_300", "kind": "lookup", "scheme": "bcht", "n": 1 << 20, "q": 300,
         "positive": 0.7, "lf": 0.9},
        # the largest lookup batch of the serving workload, on its largest table
        {"name": "lookup_1m", "kind": "lookup", "scheme": "bcht", "n": 1 << 24, "q": 1 << 20,
         "positive": 0.7, "lf": 0.9},
        # bulk lookup on a table far larger than the caches, half the keys absent
        {"name": "lookup_64m", "kind": "lookup", "scheme": "bcht", "n": 1 << 26, "q": 1 << 26,
         "positive": 0.5, "lf": 0.9},
        # a small dictionary rebuilt per request (serving builds start at 2^12 keys)
        {"name": "rebuild_5k", "kind": "rebuild", "scheme": "bcht", "n": 5000, "q": 5000,
         "positive": 0.5, "lf": 0.9},
        # the build side of a small join, an odd size below the partitioned build's default
        {"name": "rebuild_100k", "kind": "rebuild", "scheme": "bcht", "n": 100003, "q": 100003,
         "positive": 0.5, "lf": 0.9},
        # the small benchmark configuration: 2^20 keys, held in the last-level cache
        {"name": "rebuild_1m", "kind": "rebuild", "scheme": "bcht", "n": 1 << 20, "q": 1 << 20,
         "positive": 0.5, "lf": 0.9},
        # bulk build and probe of the schemes' size: the main path at full bandwidth
        {"name": "rebuild_128m", "kind": "rebuild", "scheme": "bcht", "n": 1 << 27, "q": 1 << 27,
         "positive": 0.5, "lf": 0.9},
        # 64-bit keys and values, a medium table
        {"name": "rebuild64_4m", "kind": "rebuild", "scheme": "bcht64", "n": 1 << 22, "q": 1 << 22,
         "positive": 0.5, "lf": 0.9},
        # power-of-two choices (keys never move), a medium table at a load it reaches
        {"name": "rebuild_bp2ht_1m", "kind": "rebuild", "scheme": "bp2ht", "n": 1 << 20,
         "q": 1 << 20, "positive": 0.5, "lf": 0.8},
        # two-level iceberg table, odd size, at a load every build reaches (0.85 fails for some
        # constants)
        {"name": "rebuild_iht_3m", "kind": "rebuild", "scheme": "iht", "n": 3000017, "q": 3000017,
         "positive": 0.5, "lf": 0.8},
        # many uneven tables built and queried as one batch
        {"name": "batch_256", "kind": "batch", "scheme": "bcht", "tables": 256, "lo": 10, "hi": 18,
         "positive": 0.5, "lf": 0.9},
        # serving: sixteen lookup requests answered by one coalesced launch
        {"name": "requests_16", "kind": "requests", "scheme": "bcht", "tables": 8, "lo": 12,
         "hi": 22, "count": 16, "qlo": 8, "qhi": 15, "positive": 0.7, "lf": 0.9},
    ]


def _between(rng, lo, hi):
    """A whole number between lo and hi, uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.choice(["lookup", "lookup", "rebuild", "rebuild", "rebuild", "rebuild64", "bp2ht",
                       "iht", "batch", "requests"])
    positive = rng.choice([0.1, 0.5, 0.7, 1.0])
    lf = rng.choice([0.6, 0.75, 0.8, 0.85, 0.9, 0.9])
    if what == "lookup":
        return {"kind": "lookup", "scheme": rng.choice(["bcht", "bcht", "bcht64"]),
                "n": _between(rng, 1 << 14, 1 << 26), "q": _between(rng, 1 << 8, 1 << 26),
                "positive": positive, "lf": lf}
    if what == "batch":
        hi = rng.choice([14, 16, 18])
        return {"kind": "batch", "scheme": "bcht", "tables": _between(rng, 32, 512), "lo": 10,
                "hi": hi, "positive": positive, "lf": lf}
    if what == "requests":
        return {"kind": "requests", "scheme": "bcht", "tables": rng.randint(4, 16), "lo": 12,
                "hi": 22, "count": _between(rng, 2, 48), "qlo": 8, "qhi": rng.randint(10, 18),
                "positive": positive, "lf": lf}
    scheme, top = {"rebuild": ("bcht", 1 << 26), "rebuild64": ("bcht64", 1 << 24),
                   "bp2ht": ("bp2ht", 1 << 23), "iht": ("iht", 1 << 24)}[what]
    n = _between(rng, 1 << 16 if scheme == "iht" else 1 << 12, top)
    if scheme == "bp2ht":
        lf = rng.choice([0.6, 0.7, 0.8])
    if scheme == "iht":
        lf = rng.choice([0.6, 0.7, 0.8])
    return {"kind": "rebuild", "scheme": scheme, "n": n, "q": max(1, n // rng.choice([1, 1, 2, 4])),
            "positive": positive, "lf": lf}


# ------------------------------------------------------------------ inputs

def _mix32(x):
    """A bijection of [0, 2^32) (int64 tensor), murmur3's finalizer."""
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & M32
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & M32
    return x ^ (x >> 16)


def _as32(x):
    """The low 32 bits of an int64 tensor as int32."""
    return torch.where(x >= 1 << 31, x - (1 << 32), x).to(torch.int32)


def _keys(start, index, wide):
    """Unique uniform keys of the positions index (below 2^32 - 1) of the
    stream that starts at `start`: a bijection of the position, the reserved
    all-ones key replaced by the image of a position that is never used."""
    k = _mix32((index + start) & M32)
    unused = _mix32(torch.tensor((start + M32) & M32, device=index.device))
    k = torch.where(k == M32, unused, k)
    if wide:
        # the position's image in the high half, a second image below it
        hi = torch.where(k >= 1 << 31, k - (1 << 32), k)
        return (hi << 32) | _mix32(k ^ 0x5BD1E995)
    return _as32(k)


def _pairs(gen, n, wide):
    start = int(torch.randint(0, M32, (1,), generator=gen, device="cuda"))
    keys = _keys(start, torch.arange(n, device="cuda"), wide)
    if wide:
        vals = torch.randint(-(1 << 62), 1 << 62, (n,), generator=gen, device="cuda")
    else:
        vals = torch.randint(-(1 << 31), 1 << 31, (n,), generator=gen, device="cuda",
                             dtype=torch.int32)
    return start, keys, vals


def _queries(gen, start, n, q, positive, wide):
    """q queries, each a stored key with probability `positive`, else a key
    of the same stream that is not stored; and their positions."""
    pos = torch.randint(0, n, (q,), generator=gen, device="cuda")
    if positive < 1.0:
        absent = torch.rand(q, generator=gen, device="cuda") >= positive
        pos = torch.where(absent, n + torch.arange(q, device="cuda"), pos)
    return _keys(start, pos, wide), pos


def _answers(vals, pos):
    """Values and found flags of the queries at the positions pos."""
    n = vals.numel()
    found = pos < n
    v = torch.where(found, vals[torch.where(found, pos, 0)], -1)
    return v.to(vals.dtype), found.to(torch.uint8)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _table(scheme, n, lf, seed):
    """An empty table for n pairs with constants drawn from the seed."""
    kind = "bcht" if scheme == "bcht64" else scheme
    bits = 64 if scheme == "bcht64" else 32
    p = bht.bht_params_from_seed(seed, kind, bits)
    h = p.num_hashes
    slots, more = math.ceil(n / lf), {}
    if scheme == "iht":
        # secondary slots = primary slots / 8 in buckets of 8, t = 16
        primary = math.ceil(slots * 8 / 9)
        m2 = max(1, math.ceil(primary / 64))
        slots, more = primary, {"iht_threshold": 16, "iht_secondary_b": 8, "iht_secondary_m": m2}
    return bht.Table(slots, 8 if bits == 64 else 16, kind, [p.a[i] for i in range(h)],
                     [p.b[i] for i in range(h)], key_bits=bits, rng_seed=p.rng_seed, **more)


def _sizes(case, count, lo, hi, salt):
    """`count` sizes log-uniform in [2^lo, 2^hi], fixed by the case alone."""
    rng = random.Random("%s %d %d %d %s" % (case["kind"], count, lo, hi, salt))
    return [int(2 ** rng.uniform(lo, hi)) for _ in range(count)]


class _Batch:
    """A batch handle that goes before the tables it names."""

    def __init__(self, entries):
        self.entries = entries
        self.handle = bht.bht_batch_create([(e[0].handle,) + e[1:] for e in entries])

    def __del__(self):
        bht.bht_batch_destroy(self.handle)


class _Context:
    def __init__(self, requests, items):
        self.handle = bht.bht_find_ctx_create(requests, items)

    def __del__(self):
        bht.bht_find_ctx_destroy(self.handle)


def _single(case, seed):
    gen, wide = _gen(seed), case["scheme"] == "bcht64"
    start, keys, vals = _pairs(gen, case["n"], wide)
    queries, pos = _queries(gen, start, case["n"], case["q"], case["positive"], wide)
    return keys, vals, queries, pos


def _many(case, seed):
    """Per-table pairs; queries and positions per (table, query count)."""
    gen = _gen(seed)
    sizes = _sizes(case, case["tables"], case["lo"], case["hi"], "tables")
    if case["kind"] == "batch":
        asks = [(t, n) for t, n in enumerate(sizes)]
    else:
        counts = _sizes(case, case["count"], case["qlo"], case["qhi"], "requests")
        asks = [(i % case["tables"], c) for i, c in enumerate(counts)]
    pairs = [_pairs(gen, n, False) for n in sizes]
    queries = [_queries(gen, pairs[t][0], sizes[t], c, case["positive"], False) for t, c in asks]
    return sizes, pairs, asks, queries


def _outputs(counts):
    """One value and one flag array for all requests, and each one's part."""
    total = sum(counts)
    v = torch.empty(total, dtype=torch.int32, device="cuda")
    f = torch.empty(total, dtype=torch.uint8, device="cuda")
    return v, f, list(zip(v.split(counts), f.split(counts)))


def _built(table, keys, vals):
    if table.build(keys, vals) != bht.BHT_OK:
        raise RuntimeError("the resident table did not build")
    return table


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("lookup", "rebuild"):
        keys, vals, queries, _ = _single(case, seed)
        table = _table(case["scheme"], case["n"], case["lf"], seed)
        if kind == "lookup":
            return {"kind": kind, "table": _built(table, keys, vals), "queries": queries}
        return {"kind": kind, "table": table, "keys": keys, "vals": vals, "queries": queries}
    sizes, pairs, asks, queries = _many(case, seed)
    tables = [_table("bcht", n, case["lf"], seed * 1000 + t) for t, n in enumerate(sizes)]
    values, found, parts = _outputs([c for _, c in asks])
    state = {"kind": kind, "values": values, "found": found}
    if kind == "batch":
        state["batch"] = _Batch([(tables[t], pairs[t][1], pairs[t][2], queries[i][0]) + parts[i]
                                 for i, (t, _) in enumerate(asks)])
        # a batch is captured into a graph on a stream of its own
        state["stream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        return state
    for t, (_, keys, vals) in enumerate(pairs):
        _built(tables[t], keys, vals)
    state["tables"] = tables
    state["context"] = _Context(64, 1 << 14)
    state["requests"] = [(tables[t].handle, queries[i][0]) + parts[i]
                         for i, (t, _) in enumerate(asks)]
    return state


def run(state):
    kind = state["kind"]
    if kind == "lookup":
        values, found = state["table"].find(state["queries"])
        return {"values": values, "found": found}
    if kind == "rebuild":
        status = state["table"].build(state["keys"], state["vals"])
        values, found = state["table"].find(state["queries"])
        return {"status": status, "values": values, "found": found}
    if kind == "batch":
        batch, stream = state["batch"], state["stream"]
        bht.bht_batch_run(batch.handle, stream)
        status, _ = bht.bht_batch_wait(batch.handle, len(batch.entries), stream)
        return {"status": status, "values": state["values"], "found": state["found"]}
    bht.bht_multi_find(state["context"].handle, state["requests"])
    return {"values": state["values"], "found": state["found"]}


def _lookup_bytes(buckets, bucket_bytes, q, query_bytes, value_bytes):
    """The query, its value and flag, and every bucket that some query's
    first probe names, once."""
    touched = buckets * -math.expm1(-q / buckets)
    return q * (query_bytes + value_bytes + 1) + bucket_bytes * touched


def work(case):
    word = 8 if case["scheme"] == "bcht64" else 4
    per_bucket = 8 if case["scheme"] == "bcht64" else 16

    def find(n, q):
        return _lookup_bytes(n / case["lf"] / per_bucket, 128, q, word, word)

    def build(n):
        # pairs read, every slot of the table written
        return 2 * word * n + 2 * word * n / case["lf"]

    if case["kind"] == "lookup":
        total = find(case["n"], case["q"])
    elif case["kind"] == "rebuild":
        total = build(case["n"]) + find(case["n"], case["q"])
    else:
        sizes = _sizes(case, case["tables"], case["lo"], case["hi"], "tables")
        if case["kind"] == "batch":
            total = sum(build(n) + find(n, n) for n in sizes)
        else:
            counts = _sizes(case, case["count"], case["qlo"], case["qhi"], "requests")
            total = sum(find(sizes[i % len(sizes)], c) for i, c in enumerate(counts))
    return {"bytes": float(total), "flops": 0.0}


def exact(case, seed):
    """The answers by the positions the queries were drawn from: a query at a
    stored position has that pair's value, any other is absent."""
    if case["kind"] in ("lookup", "rebuild"):
        _, vals, _, pos = _single(case, seed)
        v, f = _answers(vals, pos)
    else:
        _, pairs, asks, queries = _many(case, seed)
        got = [_answers(pairs[t][2], queries[i][1]) for i, (t, _) in enumerate(asks)]
        v, f = torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])
    out = {"values": v, "found": f}
    if case["kind"] in ("rebuild", "batch"):
        out["status"] = int(bht.BHT_OK)
    return out
