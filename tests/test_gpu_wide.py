"""Tables of 32-bit keys on either side of the lines between quotient and wide index
entries, and one table rebuilt back and forth over a line: counts, grouped counts,
pairs, intersections and erases against the oracle.  Keys repeat, so that buckets of
every length appear, long ones among them."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEED = 4711


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


def keys_of(n, V, rng):
    """n keys: half distinct, a third repeated a few times, some often, one hot."""
    k = workloads.uniform_keys(n, 32, n)
    k[: n // 3] = rng.choice(k[n // 3: n // 3 + max(1, n // 12)], n // 3)
    k[: n // 50] = rng.choice(k[-max(1, n // 2000):], n // 50)
    k[: n // 100] = k[-1]
    return rng.permutation(k)


def check(hg, t, live, V, q, keys, stable):
    exp, etot = oracle.probe_counts(live, q)
    dq = hg.to_device(q)
    c, tot = hg.hg_probe(t, dq, total=True)
    assert np.array_equal(hg.to_numpy(c, np.uint32), exp) and tot == etot
    g, _ = hg.hg_probe_ordered(t, dq, hg.PROBE_GROUPED)
    assert np.array_equal(hg.to_numpy(g, np.uint32), exp)
    few = q[np.flatnonzero(exp <= 200)[:3000]]
    fe, ft = oracle.probe_counts(live, few)
    bi, pi, ptot = hg.hg_probe_pairs(t, hg.to_device(few))
    bi, pi = hg.to_numpy(bi, np.uint32), hg.to_numpy(pi, np.uint32)
    assert ptot == ft and np.array_equal(pi, np.repeat(np.arange(few.size), fe))
    assert np.array_equal(keys[bi], few[pi])
    assert np.unique(bi.astype(np.uint64) << np.uint64(32) | pi).size == ptot
    if stable:
        assert np.all((np.diff(bi.astype(np.int64)) > 0) | (np.diff(pi.astype(np.int64)) > 0))
    b = hg.hg_build(dq, V, seed=SEED)
    ic, ia, ib, itot = hg.hg_intersect(t, b, capacity=int(etot))
    assert itot == etot and np.array_equal(hg.to_numpy(ic, np.uint32), exp)
    ia, ib = hg.to_numpy(ia, np.uint32), hg.to_numpy(ib, np.uint32)
    assert ia.size == etot and np.array_equal(keys[ia], q[ib])
    b.free()


def queries(keys, rng):
    return rng.permutation(np.concatenate([rng.choice(np.unique(keys), 3000), keys[:2000],
                                           workloads.uniform_keys(4001, 32, 9)]))


@pytest.mark.parametrize("any_order", [False, True])
@pytest.mark.parametrize("V,n", [(1, 40), (700, 350), (4095, 9000), (4096, 2048), (4096, 2049),
                                 (1 << 16, 1 << 15), ((1 << 16), (1 << 15) + 1),
                                 (65537, 98305), (65537, 98306), (1 << 18, 3 << 17),
                                 ((1 << 18) + 1, 5 * (1 << 18)), (300_000, 1_500_000),
                                 (300_000, 1_500_001)])
def test_entries_around_the_lines(hg, V, n, any_order):
    print("[case]", V, n, any_order, flush=True)
    rng = np.random.default_rng(V + n)
    k = keys_of(n, V, rng)
    q = queries(k, rng)
    t = hg.hg_build(hg.to_device(k), V, seed=SEED, any_order=any_order)
    check(hg, t, k, V, q, k, not any_order)
    gone = rng.choice(np.unique(k), min(300, np.unique(k).size // 2), replace=False)
    live = k[~np.isin(k, gone)]
    assert t.erase(hg.to_device(gone)) == k.size - live.size
    check(hg, t, live, V, q, k, not any_order)
    t.free()


def test_one_table_over_the_line_and_back(hg):
    V = 1 << 14
    t = hg.Table.create(60_000, V)
    for i, n in enumerate([8192, 60_000, 100, 8193, 0, 8000]):
        print("[case]", n, flush=True)
        rng = np.random.default_rng(n)
        if n == 0:
            t.rebuild(torch.empty(0, dtype=torch.int32, device="cuda"), V, seed=SEED)
            c, tot = hg.hg_probe(t, hg.to_device(workloads.uniform_keys(1000, 32, 2)), total=True)
            assert tot == 0 and int(c.abs().sum()) == 0
            continue
        k = keys_of(n, V, rng)
        t.rebuild(hg.to_device(k), V, seed=SEED, any_order=bool(i & 1))
        check(hg, t, k, V, queries(k, rng), k, not (i & 1))
    t.free()
