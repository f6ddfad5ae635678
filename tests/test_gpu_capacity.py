"""A table's own workspace serves builds below its capacity that need more than
the largest one does (wider bins over the same range): with an allocator that
refuses everything they succeed, also captured into a graph and replayed, and
are the oracle's tables."""
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
def test_smaller_builds_need_no_allocation(hg, kb, any_order):
    cap, V = (17_616_076, 1 << 24) if kb == 32 else (8_808_038, 1 << 24)
    n = cap - cap // 20
    print("[case]", kb, any_order, n, flush=True)
    k = workloads.uniform_keys(n, kb, 3)
    k[:n // 10] = k[0]  # a split bin
    off, ids, _ = oracle.build_table(k, V, 5, kb)
    dk = hg.to_device(k)
    other = torch.flip(dk, (0,))
    t = hg.Table.create(cap, V, kb)

    def check():
        g_off, g_ids, _ = t.export()
        g_ids = hg.to_numpy(g_ids, np.uint32)
        if any_order:
            bucket = np.repeat(np.arange(V), np.diff(off.astype(np.int64)))
            g_ids = g_ids[np.lexsort((g_ids, bucket))]
        assert np.array_equal(hg.to_numpy(g_off, np.uint32), off) and np.array_equal(g_ids, ids)

    hg.set_allocator(lambda nbytes, stream: 0, lambda ptr, stream: None)
    try:
        t.rebuild(dk, V, seed=5, any_order=any_order)
        torch.cuda.synchronize()
        check()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            t.rebuild(dk, V, seed=5, any_order=any_order)
        for _ in range(2):
            t.rebuild(other, V, seed=5)  # (as large: the host side keeps its size)
            g.replay()
            torch.cuda.synchronize()
            check()
        del g
    finally:
        hg.set_allocator()
    t.free()
