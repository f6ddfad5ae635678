"""Intersections on either side of the line between A's entries streamed and its
offsets scanned, both with quotient entries of 8 bytes: counts by edge and by input,
totals and pairs against the oracle, with repeated and hot keys, before and after keys
are erased from either side."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEED = 99


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


@pytest.mark.parametrize("V,load2,m", [(200_000, 2.99, 70_001), (200_000, 3.0, 70_001),
                                       (1 << 18, 2.0, 5), (1 << 18, 3.0, 5),
                                       (600_000, 7.99, 300_000), (600_000, 8.0, 300_000),
                                       (600_000, 8.0, 149_999), (600_000, 8.0, 150_000)])
def test_either_side_of_the_line(hg, V, load2, m):
    print("[case]", V, load2, m, flush=True)
    rng = np.random.default_rng(V + m)
    n = int(np.ceil(load2 * V / 2)) if load2 == int(load2) else int(load2 * V / 2)
    k = workloads.uniform_keys(n, 32, 1)
    k[: n // 10] = rng.choice(k[-n // 100:], n // 10)  # keys of 10 entries
    k[: n // 400] = k[-1]  # a long bucket
    k = rng.permutation(k)
    q = workloads.probe_queries(k, m, 0.6, seed=2)
    q[: m // 50] = k[-1]
    a = hg.hg_build(hg.to_device(k), V, seed=SEED)
    b = hg.hg_build(hg.to_device(q), V, seed=SEED)

    def check(live, bq):
        exp, etot = oracle.probe_counts(live, bq)
        if bq.size == q.size:  # (counts by input keep their places)
            c, _, _, tot = hg.hg_intersect(a, b)
            assert tot == etot and np.array_equal(hg.to_numpy(c, np.uint32), exp)
        else:
            _, _, _, tot = hg.hg_intersect(a, b, counts=False)
            assert tot == etot
        e, tot = hg.hg_intersect_edges(a, b)
        assert tot == etot and int(hg.to_numpy(e, np.uint32).astype(np.uint64).sum()) == etot
        assert np.array_equal(np.sort(hg.to_numpy(e, np.uint32))[-exp.size:], np.sort(exp))
        if etot < 1 << 22:
            _, ia, ib, _ = hg.hg_intersect(a, b, counts=False, capacity=int(etot))
            ia, ib = hg.to_numpy(ia, np.uint32), hg.to_numpy(ib, np.uint32)
            assert ia.size == etot and np.array_equal(k[ia], q[ib])

    check(k, q)
    gone = rng.choice(np.unique(k), 500, replace=False)
    a.erase(hg.to_device(gone))
    live = k[~np.isin(k, gone)]
    check(live, q)
    some = rng.choice(np.unique(q), max(1, m // 100), replace=False)
    b.erase(hg.to_device(some))
    check(live, q[~np.isin(q, some)])
    a.free()
    b.free()
