"""What HG_PROBE_GROUPED_UNLESS_SKEWED decides on the device: random and key-sorted
queries are grouped, queries by bucket, in runs or with a hot key keep input order.
The decision is read from a workspace block of the test's own; the counts are the
oracle's either way."""
import numpy as np
import pytest

import oracle
from paper_1907_02900_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEED, V, M, FILL = 3, 1 << 20, 1 << 19, 0x5A5A5A5A


@pytest.fixture(scope="module")
def hg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02900_amd import hg as _hg
    _hg.lib()
    return _hg


def runs(q, length, rng):
    """q with runs of equal neighbours, of that mean length."""
    new = rng.random(q.size) < 1.0 / length
    new[0] = True
    return q[np.cumsum(new) - 1]


KINDS = {  # queries, whether they are grouped
    "random": (lambda q, b, rng: q, 1),
    "sorted by key": (lambda q, b, rng: np.sort(q), 1),
    "short runs": (lambda q, b, rng: runs(q, 1.2, rng), 1),
    "by bucket": (lambda q, b, rng: q[np.argsort(b, kind="stable")], 0),
    "by range": (lambda q, b, rng: q[np.argsort(b >> 11, kind="stable")], 0),
    "runs of two": (lambda q, b, rng: runs(q, 2.0, rng), 0),
    "long runs": (lambda q, b, rng: runs(q, 300.0, rng), 0),
    "hot key": (lambda q, b, rng: np.where(rng.random(q.size) < 0.1, q[0], q), 0),
}


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("kind", list(KINDS))
def test_decision(hg, kb, kind):
    print("[case]", kb, kind, flush=True)
    rng = np.random.default_rng(kb)
    k = workloads.uniform_keys(V, kb, 1)
    q = workloads.probe_queries(k, M, 0.5, seed=2, key_bits=kb)
    make, grouped = KINDS[kind]
    q = make(q, oracle.hash_buckets(q, V, SEED, kb), rng)
    t = hg.hg_build(hg.to_device(k), V, seed=SEED, any_order=True)
    blocks = []

    def alloc(nbytes, stream):
        blocks.append(torch.full((-(-nbytes // 256) * 64,), FILL, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        return blocks[-1].data_ptr()

    hg.set_allocator(alloc, lambda ptr, stream: None)
    try:
        c, _ = hg.hg_probe_ordered(t, hg.to_device(q), hg.PROBE_GROUPED_UNLESS_SKEWED)
        torch.cuda.synchronize()
    finally:
        hg.set_allocator()
    exp, _ = oracle.probe_counts(k, q, kb)
    assert np.array_equal(hg.to_numpy(c, np.uint32), exp)
    assert len(blocks) == 1
    rows = hg.to_numpy(blocks[0], np.uint32).reshape(-1, 64)
    gate = rows[(rows[:, 1:] == FILL).all(1) & (rows[:, 0] <= 1)]
    assert gate.shape[0] == 1 and gate[0, 0] == grouped
    t.free()
