"""Searches from and to host memory at the edges of their pinned buffers (1024
query segments, 512 results), batches whose records go through pinned memory
and whose do not, and indexes built one after another on reused memory."""
import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu

FIELDS = ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi")


def _segments(n, seed, traj=True):
    rng = np.random.default_rng(seed)
    a = np.empty((8, n))
    a[0:3] = rng.uniform(0, 30, (3, n))
    a[4:7] = a[0:3] + rng.uniform(-2, 2, (3, n))
    a[3] = rng.uniform(0, 10, n)
    a[7] = a[3] + 0.8
    ids = np.arange(n, dtype=np.uint32) // 3 if traj else np.zeros(n, np.uint32)
    return trajgen.Segments(*a, traj=ids)


def _same(got, want):
    got, want = tds.sort_records(got), oracle.sort_results(want)
    assert got.size == want.size
    for f in FIELDS:
        assert np.array_equal(got[f], want[f]), f


@pytest.mark.parametrize("nq", [1, 2, 1023, 1024, 1025])
def test_host_queries(nq):
    assert torch.cuda.is_available()
    D, Q = _segments(900, 1), _segments(nq, 2)
    idx = tds.Index(D, num_bins=8)
    _same(idx.search(Q, 3.0), oracle.search(Q, D, 3.0, -np.inf, np.inf))
    idx.close()


def test_host_results_around_the_first_copy():
    D, Q = _segments(900, 3), _segments(700, 4)
    idx = tds.Index(D, num_bins=8)
    want = oracle.sort_results(oracle.search(Q, D, 4.0, -np.inf, np.inf))
    key = lambda r: r["q_seg"].astype(np.uint64) << np.uint64(32) | r["e_seg"]  # noqa: E731
    assert want.size > 513
    for cap in (0, 1, 511, 512, 513, want.size, want.size + 1):
        buf = np.zeros(max(cap, 1) + 1, tds.RESULT_DTYPE)
        st, n, _ = idx.search_raw(Q, 4.0, out_ptr=buf.ctypes.data, capacity=cap,
                                  out_on_device=False)
        assert n == want.size and st == (tds.TDS_OK if cap >= n else tds.TDS_E_OVERFLOW)
        got = tds.sort_records(buf[:min(cap, n)])
        assert np.unique(key(got)).size == got.size and np.isin(key(got), key(want)).all()
        assert buf[cap:].tobytes() == bytes(32 * (buf.size - cap))
    # few queries, few results: below the first copy's records
    q = trajgen.Segments(*[getattr(Q, f)[:40] for f in ("xs", "ys", "zs", "ts", "xe", "ye", "ze", "te")],
                         traj=Q.traj[:40])
    few = oracle.search(q, D, 2.0, -np.inf, np.inf)
    assert 0 < few.size < 512
    _same(idx.search(q, 2.0), few)
    idx.close()


@pytest.mark.parametrize("room", [900, 40000])  # with 3 requests, either side of 65536 in all
def test_batcher_records(room):
    D, Q = _segments(800, 5), _segments(300, 6)
    idx = tds.Index(D, num_bins=8)
    cut = lambda a, b: trajgen.Segments(*[getattr(Q, f)[a:b] for f in (  # noqa: E731
        "xs", "ys", "zs", "ts", "xe", "ye", "ze", "te")], traj=Q.traj[a:b])
    reqs = [(cut(0, 100), 2.0, -np.inf, np.inf), (cut(100, 101), 0.0, -np.inf, np.inf),
            (cut(101, 300), 2.5, 1.0, 7.0)]
    b = tds.Batcher(idx, max_segments=300, max_requests=3, result_capacity=3 * room)
    for _ in range(3):
        got, _, st = b.run(reqs, slice_capacity=room)
        assert st == tds.TDS_OK
        for (q, d, t0, t1), r in zip(reqs, got):
            _same(r, oracle.search(q, D, d, t0, t1))
    b.close()
    idx.close()


def test_indexes_on_reused_memory():
    Q = _segments(200, 7)
    alive = []
    for k, n in enumerate((5000, 300, 4999, 70000, 5000, 64, 70001)):
        D = _segments(n, 10 + k)
        idx = tds.Index(D, layout=("spatial", "temporal")[k % 2])
        alive.append((idx, D))
        if len(alive) > 2:
            alive.pop(0)[0].close()
        for i, d in alive:
            _same(i.search(Q, 1.5), oracle.search(Q, d, 1.5, -np.inf, np.inf))
    for i, _ in alive:
        i.close()
