"""The library's workspace pool: several threads on streams of their own get
the oracle's results from it, and what it keeps goes back to the device when
the last table is freed."""
import threading

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


def test_threads_and_streams_share_the_pool(hg):
    jobs = []
    for i in range(4):
        k = workloads.duplicate_keys(60_000 + 977 * i, 3.0, 32, seed=i)
        q = workloads.probe_queries(k, 90_001 + i, 0.5, seed=50 + i)
        jobs.append((k, q, oracle.probe_counts(k, q), hg.to_device(k), hg.to_device(q)))
    torch.cuda.synchronize()
    errors = []

    def work(i):
        k, q, (exp, etot), dk, dq = jobs[i]
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(5):
                    t = hg.hg_build(dk, 50_000, seed=i)
                    c, tot = hg.hg_probe_ordered(t, dq, hg.PROBE_GROUPED, total=True)
                    _, _, ptot = hg.hg_probe_pairs(t, dq)
                    s.synchronize()
                    assert tot == etot == ptot
                    assert np.array_equal(hg.to_numpy(c, np.uint32), exp)
                    t.free()
        except Exception as e:  # reported by the main thread
            errors.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_the_pool_is_given_back(hg):
    m = 1 << 24
    q = torch.randint(-2**31, 2**31 - 1, (m,), device="cuda", dtype=torch.int32)
    out = torch.empty(m, device="cuda", dtype=torch.int32)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    t = hg.hg_build(q, m, seed=1)
    c, tot = hg.hg_probe_ordered(t, q, hg.PROBE_GROUPED, total=True, out=out)
    torch.cuda.synchronize()
    assert torch.equal(c, out) and tot >= m
    t.free()
    torch.cuda.synchronize()
    # the table, its build's and the probe's workspace took about 700 MB
    assert torch.cuda.mem_get_info()[0] >= before - (64 << 20)


def test_probes_under_capture(hg):
    # captured without the pool: eager work between the replays uses it
    k = workloads.duplicate_keys(50_000, 2.0, 32, seed=2)
    q = workloads.probe_queries(k, 70_001, 0.5, seed=3)
    exp, _ = oracle.probe_counts(k, q)
    dq = hg.to_device(q)
    t = hg.hg_build(hg.to_device(k), 40_000, seed=4)
    for order in (hg.PROBE_INPUT_ORDER, hg.PROBE_GROUPED, hg.PROBE_GROUPED_UNLESS_SKEWED):
        out = torch.zeros(q.size, device="cuda", dtype=torch.int32)
        hg.hg_probe_ordered(t, dq, order, out=out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            hg.hg_probe_ordered(t, dq, order, out=out)
        for _ in range(4):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(hg.to_numpy(out, np.uint32), exp)
            _, tot = hg.hg_probe_ordered(t, dq, hg.PROBE_GROUPED, total=True)
            assert tot == exp.sum()
        del g
    t.free()
