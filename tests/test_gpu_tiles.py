"""Partition tiles and the grouped probe at the edges of their sizes, against
the oracle: tiles of 4096 and 8192 keys and spans of 16384 queries that end
short, runs of one range longer than a wave takes at once, and counts that do
not fit the byte they travel in.  Both key widths and orders."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [1, 4095, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385, 40961, 100003]


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("V", [3, 4097, 1 << 22])
def test_partition_tile_edges(hg, kb, V):
    for n in SIZES:
        print("[case] build", kb, V, n, flush=True)
        k = workloads.uniform_keys(n, kb, n)
        off, ids, _ = oracle.build_table(k, V, 5, kb)
        bucket = np.repeat(np.arange(V), np.diff(off.astype(np.int64)))
        for any_order in (False, True):
            t = hg.hg_build(hg.to_device(k), V, seed=5, any_order=any_order)
            g_off, g_ids, g_ek = t.export()
            torch.cuda.synchronize()
            g_ids = hg.to_numpy(g_ids, np.uint32)
            assert np.array_equal(hg.to_numpy(g_off, np.uint32), off)
            assert np.array_equal(hg.to_numpy(g_ek, k.dtype), k[g_ids])
            if any_order:
                g_ids = g_ids[np.lexsort((g_ids, bucket))]
            assert np.array_equal(g_ids, ids)
            t.free()


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("V", [1, 2, 300, 1 << 20])
@pytest.mark.parametrize("copies", [1, 254, 255, 256, 70000])
def test_grouped_counts(hg, kb, V, copies):
    # `hot` holds `copies` entries; queries: none, some or nearly all ask for it
    print("[case] probe", kb, V, copies, flush=True)
    rng = np.random.default_rng(copies + V)
    base = workloads.uniform_keys(3000, kb, 11)
    hot = base[0]
    k = rng.permutation(np.concatenate([base, np.full(copies - 1, hot)]).astype(base.dtype))
    t = hg.hg_build(hg.to_device(k), V, seed=9, any_order=True)
    for m in SIZES:
        for share in (0.0, 0.02, 0.99):
            q = np.concatenate([base, workloads.uniform_keys(m, kb, m)])
            q = rng.permutation(q)[:m]
            q[rng.random(m) < share] = hot
            exp, etot = oracle.probe_counts(k, q, kb)
            for order in (hg.PROBE_GROUPED, hg.PROBE_GROUPED_UNLESS_SKEWED):
                c, tot = hg.hg_probe_ordered(t, hg.to_device(q), order, total=True)
                assert np.array_equal(hg.to_numpy(c, np.uint32), exp) and tot == etot
    t.free()
