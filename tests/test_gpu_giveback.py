"""hg_set_allocator gives the device what the workspace pool keeps, while tables
live, and does so beside a stream capture without harm to it."""
import time

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


def test_set_allocator_empties_the_pool(hg):
    k = workloads.uniform_keys(1 << 16, 32, 1)
    t = hg.hg_build(hg.to_device(k), 1 << 16, seed=1)
    m = 1 << 25
    q = torch.randint(-2**31, 2**31 - 1, (m,), device="cuda", dtype=torch.int32)
    out = torch.empty(m, device="cuda", dtype=torch.int32)
    torch.cuda.synchronize()
    hg.set_allocator()
    time.sleep(0.5)
    free0 = torch.cuda.mem_get_info()[0]
    hg.hg_probe_ordered(t, q, hg.PROBE_GROUPED, out=out)
    torch.cuda.synchronize()
    time.sleep(0.5)
    assert free0 - torch.cuda.mem_get_info()[0] >= 11 * m - (64 << 20)  # the pool keeps it
    hg.set_allocator()
    for _ in range(100):  # (freed memory is counted some time later)
        if free0 - torch.cuda.mem_get_info()[0] < 64 << 20:
            break
        time.sleep(0.05)
    assert free0 - torch.cuda.mem_get_info()[0] < 64 << 20
    t.free()


def test_beside_a_capture(hg):
    k = workloads.duplicate_keys(50_000, 2.0, 32, seed=2)
    q = workloads.probe_queries(k, 70_001, 0.5, seed=3)
    exp, _ = oracle.probe_counts(k, q)
    dq = hg.to_device(q)
    t = hg.hg_build(hg.to_device(k), 40_000, seed=4)
    out = torch.zeros(q.size, device="cuda", dtype=torch.int32)
    hg.hg_probe_ordered(t, dq, hg.PROBE_GROUPED, out=out)  # the pool holds a block
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        hg.hg_probe(t, dq, out=out)
        hg.set_allocator()
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(hg.to_numpy(out, np.uint32), exp)
        _, tot = hg.hg_probe_ordered(t, dq, hg.PROBE_GROUPED, total=True)
        assert tot == exp.sum()
    del g
    t.free()
