"""Builds at the edges of the per-bin paths, against the oracle: one bin at the
light kernel's capacity, heavy and split bins next to each other whose long
buckets lie at the bins' ends, slices that end short, and the largest build
whose heavy bins are not split.  Both key widths, stable and any order, with
and without the probe index."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEED = 77


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


def dt(kb):
    return np.uint64 if kb == 64 else np.uint32


def check(hg, k, V, kb):
    off, ids, ek = oracle.build_table(k, V, SEED, kb)
    q = workloads.probe_queries(k, 20000, 0.5, seed=3, key_bits=kb)
    exp, etot = oracle.probe_counts(k, q, kb)
    bucket = np.repeat(np.arange(V), np.diff(off.astype(np.int64)))
    for any_order in (False, True):
        for index in (True, False):
            t = hg.hg_build(hg.to_device(k), V, seed=SEED, any_order=any_order, index=index)
            g_off, g_ids, g_ek = t.export()
            torch.cuda.synchronize()
            g_ids, g_ek = hg.to_numpy(g_ids, np.uint32), hg.to_numpy(g_ek, dt(kb))
            assert np.array_equal(hg.to_numpy(g_off, np.uint32), off)
            assert np.array_equal(g_ek, k[g_ids])
            if any_order:
                g_ids = g_ids[np.lexsort((g_ids, bucket))]
            assert np.array_equal(g_ids, ids)
            c, tot = hg.hg_probe(t, hg.to_device(q), counts=True, total=True)
            assert np.array_equal(hg.to_numpy(c, np.uint32), exp) and tot == etot
            t.free()


@pytest.mark.parametrize("kind", ["uniform", "dup100", "equal"])
@pytest.mark.parametrize("V", [1, 100, 4096])
@pytest.mark.parametrize("kb,n", [(32, 1), (32, 33), (32, 4607), (32, 4608), (32, 4609),
                                  (64, 1), (64, 33), (64, 3071), (64, 3072), (64, 3073)])
def test_one_bin_at_capacity(hg, kb, n, V, kind):
    print("[case]", kb, n, V, kind, flush=True)
    k = {"uniform": lambda: workloads.uniform_keys(n, kb, 9),
         "dup100": lambda: workloads.duplicate_keys(n, 100.0, kb, 9),
         "equal": lambda: np.full(n, 3, dt(kb))}[kind]()
    check(hg, k, min(V, 2048) if kb == 64 else V, kb)


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("n", [(1 << 17) - 1, 1 << 17, (1 << 17) + 1, 200001])
@pytest.mark.parametrize("big", [16383, 16384, 16385, 32769, 49153])
def test_neighbouring_oversize_bins(hg, kb, n, big):
    # 2^14 keys a slice above 2^17 keys, no slices up to it
    print("[case]", kb, n, big, flush=True)
    V = 1 << 16
    rng = np.random.default_rng(n + big)
    pool = workloads.uniform_keys(1 << 21, kb, 4)
    h = oracle.hash_buckets(pool, V, SEED, kb)
    parts = []
    # the last and the first bucket of neighbouring bins at every bin width
    for lo, hi, count, distinct in [((1 << 14) - 1, 1 << 14, big, 1),
                                    (1 << 14, (1 << 14) + 2048, big, 5000),
                                    ((1 << 14) + 4095, (1 << 14) + 4096, 700, 12),
                                    (V - 1, V, 6000, 2)]:
        have = pool[(h >= lo) & (h < hi)][:distinct]
        parts.append(rng.choice(have, count) if distinct > 1 else np.repeat(have, count))
    k = np.concatenate(parts)[:n]
    k = np.concatenate([k, workloads.uniform_keys(n - k.size, kb, 8)])
    check(hg, rng.permutation(k), V, kb)


@pytest.mark.parametrize("n", [(1 << 24) - 1, 1 << 24])
def test_split_bins_with_and_without_their_own_histogram_kernel(hg, n):
    print("[case]", n, flush=True)
    rng = np.random.default_rng(n)
    k = workloads.uniform_keys(n, 32, 4)
    k[rng.random(n) < 0.2] = 7  # one split bin of about 200 slices
    k[rng.random(n) < 0.001] = 9  # and an oversize one
    V = 1 << 24
    off, ids, ek = oracle.build_table(k, V, SEED, 32)
    t = hg.hg_build(hg.to_device(k), V, seed=SEED)
    g_off, g_ids, g_ek = t.export()
    torch.cuda.synchronize()
    assert np.array_equal(hg.to_numpy(g_off, np.uint32), off)
    assert np.array_equal(hg.to_numpy(g_ids, np.uint32), ids)
    assert np.array_equal(hg.to_numpy(g_ek, np.uint32), ek)
    c, tot = hg.hg_probe(t, hg.to_device(k[:50000]), counts=True, total=True)
    exp, etot = oracle.probe_counts(k, k[:50000], 32)
    assert np.array_equal(hg.to_numpy(c, np.uint32), exp) and tot == etot
    t.free()
