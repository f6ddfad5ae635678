"""The probe index's entry formats on the GPU: buckets of chosen lengths --
held whole in the entry, at and past its capacity, past the lane-built
length, long ones of one key, of a dominant key and of many keys -- over hash
ranges that give 4- and 8-byte entries.  Counts, pairs and intersections equal
the oracle's, before and after an erase."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


def unfmix32(x):
    """Inverse of the MurmurHash3 32-bit finaliser."""
    x = x.astype(np.uint64)
    m = np.uint64(0xFFFFFFFF)
    x ^= x >> np.uint64(16)
    x = x * np.uint64(pow(0xC2B2AE35, -1, 1 << 32)) & m
    x ^= (x >> np.uint64(13)) ^ (x >> np.uint64(26))
    x = x * np.uint64(pow(0x85EBCA6B, -1, 1 << 32)) & m
    x ^= x >> np.uint64(16)
    return x.astype(np.uint32)


def chosen_keys(V, seed, lens, rng):
    """Keys of chosen buckets: per length one bucket of distinct keys, one of
    a single key and one of a dominant key with others, and uniform keys
    around them; and queries for every kind of answer."""
    qmax = 0xFFFFFFFF // V
    keys, queries = [workloads.uniform_keys(2000, 32, 5)], [workloads.uniform_keys(3000, 32, 6)]
    b = 0
    for s in lens:
        for kind in range(3):
            b += max(1, V // 400)
            h = b % V
            top = (0xFFFFFFFF - h) // V  # quotients of this bucket: 0 .. top
            span = min(top + 1, 1 << 16)
            if kind == 0:
                q = rng.permutation(span)[:s]
            elif kind == 1:
                q = np.full(s, rng.integers(0, span))
            else:
                q = rng.integers(0, span, s)
                q[rng.random(s) < 0.8] = q[0] if s else 0
            keys.append(unfmix32(np.uint64(h) + q.astype(np.uint64) * np.uint64(V)) ^ np.uint32(seed))
            near = np.unique(np.concatenate([q, rng.integers(0, span, 40)])).astype(np.uint64)
            queries.append(unfmix32(np.uint64(h) + near * np.uint64(V)) ^ np.uint32(seed))
    assert qmax >= 0
    return rng.permutation(np.concatenate(keys)), rng.permutation(np.concatenate(queries))


@pytest.mark.parametrize("any_order", [False, True])
@pytest.mark.parametrize("V", [1, 3, 64, 1000, 1 << 16, (1 << 20) + 7, 1 << 23, (1 << 25) + 3,
                               1 << 26])
def test_entry_formats_match_oracle(hg, V, any_order):
    rng = np.random.default_rng(V + any_order)
    seed = 0x9E3779B9 if V % 2 else 12345
    lens = list(range(0, 20)) + [31, 32, 33, 34, 63, 64, 65, 97, 98, 200, 700]
    keys, queries = chosen_keys(V, seed, lens, rng)
    t = hg.hg_build(hg.to_device(keys), V, seed=seed, any_order=any_order)

    def check(live):
        c, tot = hg.hg_probe(t, hg.to_device(queries), total=True)
        oc, otot = oracle.probe_counts(live, queries)
        assert np.array_equal(hg.to_numpy(c, np.uint32), oc) and tot == otot
        g, _ = hg.hg_probe_ordered(t, hg.to_device(queries), hg.PROBE_GROUPED)
        assert np.array_equal(hg.to_numpy(g, np.uint32), oc)
        bi, pi, ptot = hg.hg_probe_pairs(t, hg.to_device(queries))
        bi, pi = hg.to_numpy(bi, np.uint32), hg.to_numpy(pi, np.uint32)
        assert ptot == otot and np.array_equal(keys[bi], queries[pi])
        assert np.array_equal(pi, np.repeat(np.arange(queries.size), oc))
        assert np.unique(bi.astype(np.uint64) << np.uint64(32) | pi).size == ptot
        if not any_order:  # ids ascend inside a query
            assert np.all((np.diff(bi.astype(np.int64)) > 0) | (np.diff(pi.astype(np.int64)) > 0))
        u = hg.hg_build(hg.to_device(queries), V, seed=seed)
        ic, _, _, itot = hg.hg_intersect(t, u)
        assert itot == otot and np.array_equal(hg.to_numpy(ic, np.uint32), oc)

    check(keys)
    gone = rng.choice(np.unique(keys), 400, replace=False)
    live = keys[~np.isin(keys, gone)]
    assert t.erase(hg.to_device(gone)) == keys.size - live.size
    check(live)
