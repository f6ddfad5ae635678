"""Builds whose bins nearly all list long buckets of many keys -- more bins than
the kernel that sorts them has workgroups -- beside an oversize and a split bin,
against the oracle.  Both key widths and orders."""
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


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("any_order", [False, True])
@pytest.mark.parametrize("V,bins", [(1000, 1000), (4096, 4096), (4100, 2050)])
def test_every_bin_lists_long_buckets(hg, kb, any_order, V, bins):
    print("[case]", kb, any_order, V, bins, flush=True)
    rng = np.random.default_rng(V + kb)
    k = workloads.uniform_keys(90 * V, kb, 3)
    k = np.concatenate([k, np.repeat(k[:1], 6000), np.repeat(k[7:8], 40000)])
    k = np.concatenate([k, workloads.duplicate_keys(max(0, 200_000 - k.size), 3.0, kb, 5)])
    k = rng.permutation(k)
    assert k.size > 1 << 17
    off, ids, _ = oracle.build_table(k, V, 5, kb)
    t = hg.hg_build(hg.to_device(k), V, seed=5, bins=bins, any_order=any_order)
    g_off, g_ids, _ = t.export()
    g_ids = hg.to_numpy(g_ids, np.uint32)
    if any_order:
        bucket = np.repeat(np.arange(V), np.diff(off.astype(np.int64)))
        g_ids = g_ids[np.lexsort((g_ids, bucket))]
    assert np.array_equal(hg.to_numpy(g_off, np.uint32), off) and np.array_equal(g_ids, ids)
    q = np.concatenate([np.unique(k)[:100_000], workloads.uniform_keys(50_000, kb, 9)])
    c, tot = hg.hg_probe(t, hg.to_device(q), total=True)
    exp, etot = oracle.probe_counts(k, q, kb)
    assert np.array_equal(hg.to_numpy(c, np.uint32), exp) and tot == etot
    bi, pi, ptot = hg.hg_probe_pairs(t, hg.to_device(q[:50_000]))
    ob, op, ototal = oracle.probe_pairs(k, q[:50_000], kb)
    assert ptot == ototal and np.array_equal(hg.to_numpy(pi, np.uint32), op)
    if not any_order:
        assert np.array_equal(hg.to_numpy(bi, np.uint32), ob)
    t.free()
