"""The flag that sends the rare path's first kernel through the bins held in
LDS comes from the per-bin kernel alone: a build whose long buckets all lie in
oversize bins leaves it clear, one with a long bucket of many keys in an LDS bin
sets it, and both build the oracle's table.  (Set by a workgroup of the kernel
that reads it, its waves would take different numbers of barriers.)  The
counters are found in a workspace block of the test's own."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEED = 77
FILL = 0x5A5A5A5A


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


def counters(words):
    """The six device counters: the one 256-byte block of the workspace with six
    small words and nothing written behind them."""
    rows = words[:words.size // 64 * 64].reshape(-1, 64)
    hit = rows[(rows[:, 6:] == FILL).all(1) & (rows[:, :6] < 1000).all(1)]
    assert hit.shape[0] == 1, hit[:, :8]
    return hit[0, :6]


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("any_order", [False, True])
@pytest.mark.parametrize("n", [100_000, 200_001])  # one kernel; slices as well
@pytest.mark.parametrize("listed", [False, True])
def test_only_lds_bins_raise_the_flag(hg, kb, any_order, n, listed):
    print("[case]", kb, any_order, n, listed, flush=True)
    V = 1 << 16
    rng = np.random.default_rng(n)
    pool = workloads.uniform_keys(1 << 24 if listed else 1 << 16, kb, 4)
    h = oracle.hash_buckets(pool, V, SEED, kb)
    parts = [np.repeat(pool[h == h[0]][:1], 7000)]  # an oversize bin, one long bucket
    if listed:  # 150 keys twice in one bucket, its bin far from the other
        b = (int(h[0]) + V // 2) % V
        parts.append(np.repeat(pool[h == b][:150], 2))
        assert parts[1].size == 300
    k = np.concatenate(parts)
    k = rng.permutation(np.concatenate([k, workloads.uniform_keys(n - k.size, kb, 8)]))
    blocks = []

    def alloc(nbytes, stream):
        blocks.append(torch.full((-(-nbytes // 256) * 64,), FILL, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        return blocks[-1].data_ptr()

    hg.set_allocator(alloc, lambda ptr, stream: None)
    try:
        t = hg.hg_build(hg.to_device(k), V, seed=SEED, any_order=any_order)
        torch.cuda.synchronize()
    finally:
        hg.set_allocator()
    assert len(blocks) == 1
    ctr = counters(hg.to_numpy(blocks[0], np.uint32))
    assert ctr[0] == 1 and ctr[5] == listed  # oversize bins, the flag
    off, ids, _ = oracle.build_table(k, V, SEED, kb)
    g_off, g_ids, _ = t.export()
    g_ids = hg.to_numpy(g_ids, np.uint32)
    if any_order:
        bucket = np.repeat(np.arange(V), np.diff(off.astype(np.int64)))
        g_ids = g_ids[np.lexsort((g_ids, bucket))]
    assert np.array_equal(hg.to_numpy(g_off, np.uint32), off) and np.array_equal(g_ids, ids)
    q = np.concatenate([k[:20000], workloads.uniform_keys(20000, kb, 9)])
    c, tot = hg.hg_probe(t, hg.to_device(q), total=True)
    exp, etot = oracle.probe_counts(k, q, kb)
    assert np.array_equal(hg.to_numpy(c, np.uint32), exp) and tot == etot
    t.free()
