"""Workloads of the HashGraph path as a program runs them, for timing.

Each case is a dict of plain values.  `prepare` makes what the program holds
before the call (device arrays, a preallocated or built table, a plan), `run`
is one pass through the binding's public calls, and `exact` gives the same
outputs in plain torch.  Kinds of case:

  build       rebuild of a preallocated table in the stable layout
  step        rebuild of a preallocated table, then match counts of queries
  probe       match counts of queries against a built table
  pairs       the matching (build id, query id) pairs
  intersect   Alg. 3 on two built tables: counts by input index and the total
  batch       build and probe of many tables in one graph launch
  collection  match counts of many set pairs of a collection built once
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1907_02900_amd import hg

ZIPF_DISTINCT = 1 << 24
MASK32 = 0xFFFFFFFF


def listed():
    return [
        # the benchmark's step: 2^28 uniform keys, load 1, as many queries
        dict(name="step_2p28", kind="step", n=1 << 28, m=1 << 28, range=1 << 28, bits=32,
             keys="uniform", any_order=True),
        # the hash-range sweep's dense end: four keys per bucket
        dict(name="step_load4", kind="step", n=1 << 27, m=1 << 27, range=1 << 25, bits=32,
             keys="uniform", any_order=True),
        # 64-bit keys in the stable layout, the sweep's size
        dict(name="step_u64", kind="step", n=1 << 27, m=1 << 27, range=1 << 27, bits=64,
             keys="uniform", any_order=False),
        # a skewed join: Zipf(1.2) on both sides, stable layout
        dict(name="step_zipf", kind="step", n=1 << 26, m=1 << 27, range=1 << 26, bits=32,
             keys="zipf", zipf=1.2, any_order=False),
        # the smallest builds of a request stream: launches count
        dict(name="build_small", kind="build", n=1500, range=1500, bits=32, keys="uniform"),
        # an ordinary request's build, odd sizes
        dict(name="build_mid", kind="build", n=300_007, range=300_007, bits=32, keys="uniform"),
        # a small request's probe of a medium table
        dict(name="probe_small", kind="probe", n=100_003, m=1500, range=100_003, bits=32,
             keys="uniform"),
        # a large request's probe of the stream's largest table
        dict(name="probe_mid", kind="probe", n=1 << 24, m=3_000_001, range=1 << 24, bits=32,
             keys="uniform"),
        # a join that needs the pairs themselves
        dict(name="pairs", kind="pairs", n=1 << 24, m=1 << 22, range=1 << 24, bits=32,
             keys="balanced", appearances=1),
        # Probe-New's intersection at the paper's 32M keys
        dict(name="intersect", kind="intersect", n=1 << 25, m=1 << 25, range=1 << 25, bits=32,
             keys="uniform"),
        # thousands of tables of uneven size, one graph launch
        dict(name="batch_4096", kind="batch", tables=4096, lo=8.0, hi=20.0, shape=7, bits=32),
        # build once, intersect many: rows of a sparse matrix
        dict(name="collection", kind="collection", sets=1 << 20, pairs=1 << 24, mean=32.0,
             key_range=1 << 20, shape=31, bits=32),
    ]


def _log(rng, lo, hi):
    return int(2.0 ** rng.uniform(lo, hi))


def draw(rng):
    kind = rng.choice(["build", "build", "step", "step", "probe", "probe", "pairs", "intersect",
                       "batch", "collection"])
    bits = rng.choice([32, 32, 32, 64])
    if kind == "batch":
        return dict(kind=kind, tables=_log(rng, 4, 10), lo=8.0, hi=round(rng.uniform(14, 20), 2),
                    shape=rng.randrange(1 << 20), bits=bits)
    if kind == "collection":
        return dict(kind=kind, sets=_log(rng, 10, 19), pairs=_log(rng, 12, 22),
                    mean=round(rng.uniform(8, 64), 1), key_range=1 << rng.randrange(16, 24),
                    shape=rng.randrange(1 << 20), bits=bits)
    top = 24 if kind == "pairs" else 26
    n = _log(rng, 10, top)
    load = rng.choice([0.25, 0.5, 1.0, 1.0, 1.0, 2.0, 4.0])
    c = dict(kind=kind, n=n, range=max(1, int(n / load)), bits=bits,
             keys=rng.choice(["uniform", "uniform", "sequence", "duplicates", "zipf"]))
    if rng.random() < 0.3:  # power-of-two ranges are common in practice
        c["range"] = 1 << max(0, c["range"].bit_length() - 1)
    if c["keys"] == "duplicates":
        c["appearances"] = rng.choice([2, 4, 8, 16, 32])
    if c["keys"] == "zipf":
        c["bits"] = 32
        c["zipf"] = rng.choice([0.8, 1.2, 1.5])
        if kind == "intersect":  # both sides skewed: kept to the mildest law
            c["zipf"] = 0.8
    if kind == "pairs":  # every key repeated as often, so that the total is known
        for k in ("zipf", "appearances"):
            c.pop(k, None)
        c["keys"], c["appearances"] = "balanced", rng.choice([1, 1, 2, 4, 8])
        c["n"] = max(1, n // c["appearances"]) * c["appearances"]
    if kind != "build":
        c["m"] = _log(rng, 10, top)
    if kind == "step":
        c["any_order"] = rng.random() < 0.5
    return c


# ----------------------------------------------------------------- inputs ---

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _dtype(bits):
    return torch.int64 if bits == 64 else torch.int32


def _uniform(n, bits, g):
    if bits == 64:
        return torch.randint(-(1 << 63), (1 << 63) - 1, (n,), dtype=torch.int64, device="cuda",
                             generator=g)
    return torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int32, device="cuda", generator=g)


def _zipf(n, s, mult, add, g):
    r = torch.arange(1, ZIPF_DISTINCT + 1, dtype=torch.float64, device="cuda")
    cdf = torch.cumsum(r.pow(-s), 0)
    cdf /= cdf[-1].clone()
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    for a in range(0, n, 1 << 25):
        b = min(n, a + (1 << 25))
        u = torch.rand(b - a, dtype=torch.float64, device="cuda", generator=g)
        rank = torch.searchsorted(cdf, u, right=True).clamp_(max=ZIPF_DISTINCT - 1)
        out[a:b] = ((rank * mult + add) & MASK32).to(torch.int32)
    return out


def _keys(case, seed):
    """Build keys, and queries (or B's keys): about half of them drawn from
    the build keys (Zipf: all from the same law)."""
    g = _gen(seed)
    n, m, bits = case["n"], case.get("m", 0), case["bits"]
    if case["keys"] == "zipf":
        mult, add = (2 * (seed * 7919 % (1 << 30)) + 1), seed * 104729 % (1 << 32)
        return (_zipf(n, case["zipf"], mult, add, g),
                _zipf(m, case["zipf"], mult, add, g) if m else None)
    if case["keys"] == "balanced":
        # distinct values, each in the table equally often; half of the
        # queries (to the unit) hit
        distinct = n // case["appearances"]
        mult, add = 2 * (seed * 7919 % (1 << 29)) + 0x3C6EF373, seed * 104729 % (1 << 32)
        of = lambda i: (i * mult + add).to(_dtype(bits))  # noqa: E731
        keys = of(torch.randperm(n, device="cuda", generator=g) % distinct)
        pick = torch.randint(0, distinct, (m,), device="cuda", generator=g)
        miss = torch.randint(distinct, 1 << 31, (m,), device="cuda", generator=g)
        hit = torch.randperm(m, device="cuda", generator=g) < m // 2
        return keys, of(torch.where(hit, pick, miss))
    if case["keys"] == "uniform":
        keys = _uniform(n, bits, g)
    elif case["keys"] == "sequence":
        first = seed % 1000 + 1
        keys = torch.arange(first, first + n, dtype=torch.int64, device="cuda").to(_dtype(bits))
    else:
        keys = torch.randint(1, max(1, n // case["appearances"]) + 1, (n,), dtype=_dtype(bits),
                             device="cuda", generator=g)
    if not m:
        return keys, None
    q = _uniform(m, bits, g)
    pick = torch.randint(0, n, (m,), device="cuda", generator=g)
    hit = torch.rand(m, device="cuda", generator=g) < 0.5
    return keys, torch.where(hit, keys[pick], q)


def _batch_sizes(case):
    u = np.random.default_rng(case["shape"]).uniform(case["lo"], case["hi"], case["tables"])
    return np.floor(np.exp2(u)).astype(np.int64)


def _batch_arrays(case, seed):
    g = _gen(seed)
    sizes = _batch_sizes(case)
    tot = int(sizes.sum())
    base = np.concatenate([[0], np.cumsum(sizes)])
    sz = torch.from_numpy(sizes).cuda()
    start = torch.repeat_interleave(torch.from_numpy(base[:-1]).cuda(), sz, output_size=tot)
    size = torch.repeat_interleave(sz, sz, output_size=tot)
    keys = _uniform(tot, case["bits"], g)
    q = _uniform(tot, case["bits"], g)
    pick = (torch.rand(tot, dtype=torch.float64, device="cuda", generator=g) * size).long()
    hit = torch.rand(tot, device="cuda", generator=g) < 0.5
    return sizes, base, keys, torch.where(hit, keys[start + pick], q)


def _set_offsets(case):
    r = np.random.default_rng(case["shape"])
    scale = (case["mean"] - 1.0) * 0.5
    sizes = np.minimum(1 + np.floor(r.pareto(1.5, case["sets"]) * scale), 1 << 16)
    return np.concatenate([[0], np.cumsum(sizes.astype(np.int64))])


def _collection_arrays(case, seed):
    g = _gen(seed)
    off = _set_offsets(case)
    keys = torch.randint(0, case["key_range"], (int(off[-1]),), dtype=_dtype(case["bits"]),
                         device="cuda", generator=g)
    pairs = torch.randint(0, case["sets"], (case["pairs"], 2), dtype=torch.int32, device="cuda",
                          generator=g)
    return torch.from_numpy(off.astype(np.int32)).cuda(), keys, pairs


class _View:
    """A library-owned device array, for torch.as_tensor without a copy."""

    def __init__(self, owner, ptr, count, bits):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (int(count),), "typestr": "<i%d" % (bits // 8),
                                         "data": (int(ptr), False), "version": 2}


def _view(table, ptr, count, bits):
    return torch.as_tensor(_View(table, ptr, count, bits), device="cuda")


def _seed64(seed):
    return int(seed) * 0x9E3779B97F4A7C15 & (2 ** 64 - 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sizes, base, keys, q = _batch_arrays(case, seed)
        V = int(sizes.sum())
        off = torch.empty(V + len(sizes), dtype=torch.int32, device="cuda")
        ids = torch.empty(V, dtype=torch.int32, device="cuda")
        ekeys = torch.empty_like(keys)
        counts = torch.empty(V, dtype=torch.int32, device="cuda")
        tables = []
        for i, s in enumerate(sizes.tolist()):
            a = int(base[i])
            tables.append(dict(keys=keys[a:a + s], queries=q[a:a + s], hash_range=s, seed=i,
                               offsets=off[a + i:a + i + s + 1], ids=ids[a:a + s],
                               ekeys=ekeys[a:a + s], counts=counts[a:a + s]))
        plan = hg.Batch(tables, key_bits=case["bits"])
        return dict(kind=kind, plan=plan, out=dict(offsets=off, ids=ids, ekeys=ekeys,
                                                   counts=counts))
    if kind == "collection":
        off, keys, pairs = _collection_arrays(case, seed)
        return dict(kind=kind, coll=hg.Collection(keys, off, seed=_seed64(seed)), pairs=pairs)
    keys, q = _keys(case, seed)
    n, V, bits, s64 = case["n"], case["range"], case["bits"], _seed64(seed)
    st = dict(kind=kind, keys=keys, queries=q, range=V, seed=s64)
    if kind in ("build", "step"):
        st["table"] = t = hg.Table.create(n, V, bits)
        i = t.info()
        st["any_order"] = bool(case.get("any_order"))
        st["out"] = dict(offsets=_view(t, i.d_offsets, V + 1, 32))
        if not st["any_order"]:  # (else the order inside a bucket is unspecified)
            st["out"]["ids"] = _view(t, i.d_ids, n, 32)
            st["out"]["keys"] = _view(t, i.d_keys, n, bits)
        if kind == "step":
            st["out"]["counts"] = torch.empty(q.numel(), dtype=torch.int32, device="cuda")
        return st
    st["table"] = hg.hg_build(keys, V, seed=s64)
    if kind == "probe":
        st["counts"] = torch.empty(q.numel(), dtype=torch.int32, device="cuda")
    elif kind == "pairs":
        st["capacity"] = hg.hg_probe(st["table"], q, counts=False, total=True)[1]
    elif kind == "intersect":
        st["other"] = hg.hg_build(q, V, seed=s64)
    return st


def run(state):
    kind = state["kind"]
    if kind in ("build", "step"):
        t = state["table"].rebuild(state["keys"], state["range"], state["seed"],
                                   any_order=state["any_order"])
        if kind == "step":
            hg.hg_probe(t, state["queries"], out=state["out"]["counts"])
        return state["out"]
    if kind == "probe":
        return hg.hg_probe(state["table"], state["queries"], out=state["counts"])[0]
    if kind == "pairs":
        return hg.hg_probe_pairs(state["table"], state["queries"], capacity=state["capacity"])
    if kind == "intersect":
        counts, _, _, total = hg.hg_intersect(state["table"], state["other"])
        return counts, total
    if kind == "batch":
        state["plan"].run()
        return state["out"]
    return state["coll"].intersect(state["coll"], state["pairs"])


def work(case):
    """Inputs read once and outputs written once; the part of a table that
    queries can reach is read at most whole."""
    kind, kb = case["kind"], case["bits"] // 8
    if kind == "batch":
        n = int(_batch_sizes(case).sum())
        return dict(bytes=n * kb + n * (kb + 4) + 4 * n + n * kb + 4 * n, flops=0)
    if kind == "collection":
        off = _set_offsets(case)
        n, S = float(off[-1]), case["sets"]
        sizes = np.sort(np.diff(off))  # mean of the smaller set of a random pair
        walked = float(np.sum(sizes * (2.0 * (S - np.arange(S)) - 1.0)) / (float(S) * S))
        table = n * kb + 4 * n
        look = case["pairs"] * walked * (2 * kb + 8)
        return dict(bytes=case["pairs"] * 16 + min(2 * table, look), flops=0)
    n, V, m = case["n"], case["range"], case.get("m", 0)
    build = n * kb + n * (kb + 4) + 4 * (V + 1)
    reach = min(4 * (V + 1) + n * kb, m * (8 + kb * math.ceil(n / V)))
    probe = m * kb + reach + 4 * m
    if kind == "build":
        return dict(bytes=build, flops=0)
    if kind == "step":
        return dict(bytes=build + m * kb + 4 * m, flops=0)
    if kind == "probe":
        return dict(bytes=probe, flops=0)
    if kind == "pairs":
        hits = (m // 2) * case["appearances"]
        return dict(bytes=m * kb + reach + 4 * hits + 8 * hits, flops=0)
    return dict(bytes=m * (kb + 4) + reach + 4 * m, flops=0)


# ----------------------------------------------- the same in plain torch ---

def _shr(x, s):
    return (x >> s) & ((1 << (64 - s)) - 1)


def _signed(c):
    return c - (1 << 64) if c >= 1 << 63 else c


def _bucket(keys, V, seed):
    """Eq. 1: fmix(key ^ seed) mod V, in 64-bit integers."""
    if keys.dtype == torch.int32:
        x = (keys.long() & MASK32) ^ (seed & MASK32)
        x = ((x ^ (x >> 16)) * 0x85EBCA6B) & MASK32
        x = ((x ^ (x >> 13)) * 0xC2B2AE35) & MASK32
        return (x ^ (x >> 16)) % V
    x = keys ^ _signed(seed)
    x = (x ^ _shr(x, 33)) * _signed(0xFF51AFD7ED558CCD)
    x = (x ^ _shr(x, 33)) * _signed(0xC4CEB9FE1A85EC53)
    x = x ^ _shr(x, 33)
    return (_shr(x, 1) % V * 2 + (x & 1)) % V  # unsigned x mod V


def _offsets(h, V):
    off = torch.zeros(V + 1, dtype=torch.int64, device=h.device)
    off[1:] = torch.cumsum(torch.bincount(h, minlength=V), 0)
    return off.to(torch.int32)


def _exact_table(keys, V, seed):
    h = _bucket(keys, V, seed)
    ids = torch.sort(h, stable=True).indices
    return dict(offsets=_offsets(h, V), ids=ids.to(torch.int32), keys=keys[ids])


def _exact_range(keys_sorted, q):
    lo = torch.searchsorted(keys_sorted, q)
    return lo, torch.searchsorted(keys_sorted, q, right=True) - lo


def _exact_counts(keys, q):
    return _exact_range(torch.sort(keys).values, q)[1].to(torch.int32)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sizes, base, keys, q = _batch_arrays(case, seed)
        parts = dict(offsets=[], ids=[], ekeys=[], counts=[])
        for i, s in enumerate(sizes.tolist()):
            k = keys[int(base[i]):int(base[i]) + s]
            t = _exact_table(k, s, i)
            parts["offsets"].append(t["offsets"])
            parts["ids"].append(t["ids"])
            parts["ekeys"].append(t["keys"])
            parts["counts"].append(_exact_counts(k, q[int(base[i]):int(base[i]) + s]))
        return {k: torch.cat(v) for k, v in parts.items()}
    if kind == "collection":
        return _exact_collection(case, seed)
    keys, q = _keys(case, seed)
    V, s64 = case["range"], _seed64(seed)
    if kind in ("build", "step"):
        if case.get("any_order"):
            out = dict(offsets=_offsets(_bucket(keys, V, s64), V))
        else:
            out = _exact_table(keys, V, s64)
        if kind == "step":
            out["counts"] = _exact_counts(keys, q)
        return out
    if kind == "pairs":
        ks, order = torch.sort(keys, stable=True)
        lo, cnt = _exact_range(ks, q)
        tot = int(cnt.sum())
        j = torch.repeat_interleave(torch.arange(q.numel(), device="cuda"), cnt, output_size=tot)
        first = torch.cumsum(cnt, 0) - cnt
        at = lo[j] + torch.arange(tot, device="cuda") - first[j]
        return order[at].to(torch.int32), j.to(torch.int32), tot
    counts = _exact_counts(keys, q)
    if kind == "probe":
        return counts
    return counts, int(counts.long().sum())


def _exact_collection(case, seed):
    off, keys, pairs = _collection_arrays(case, seed)
    off = off.long()
    size = off[1:] - off[:-1]
    # every (set, key) as one number; keys are below 2^24
    owner = torch.repeat_interleave(torch.arange(case["sets"], device="cuda"), size,
                                    output_size=keys.numel())
    both = torch.sort(owner * (1 << 24) + keys.long()).values
    counts = torch.zeros(case["pairs"], dtype=torch.int64, device="cuda")
    for a in range(0, case["pairs"], 1 << 20):
        p = pairs[a:a + (1 << 20)].long()
        i, j = p[:, 0], p[:, 1]
        swap = size[i] > size[j]
        i, j = torch.where(swap, j, i), torch.where(swap, i, j)
        w = size[i]
        row = torch.repeat_interleave(torch.arange(p.shape[0], device="cuda"), w)
        first = torch.cumsum(w, 0) - w
        k = keys[off[i][row] + torch.arange(row.numel(), device="cuda") - first[row]].long()
        _, c = _exact_range(both, j[row] * (1 << 24) + k)
        counts[a:a + (1 << 20)].index_add_(0, row, c)
    return counts, int(counts.sum())
