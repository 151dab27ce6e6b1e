"""Candidates per work item chosen by the number of work items (chunk = 0).

One bin holds every entry and every query segment covers it, so the work items
are (query segments / 64, rounded up) x (candidates / chunk, rounded up), and
the number aimed at is 6 per workgroup of the distance kernel: the cases lie on
both sides of it, and at the smallest and the largest chunk.
"""
import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu


def _segments(n, seed):
    """n segments, all over [0, 1] in time, in a box where a segment has about 60 within 4."""
    rng = np.random.default_rng(seed)
    a = np.empty((8, n))
    a[0:3] = rng.uniform(0, 40, (3, n))
    a[4:7] = a[0:3] + rng.uniform(-1, 1, (3, n))
    a[3], a[7] = 0.0, 1.0
    return trajgen.Segments(*a, traj=np.arange(n, dtype=np.uint32))


N = 16384  # candidates: 4 chunks of 4096, 128 of 128


@pytest.mark.parametrize("prec,groups,blocks,chunk", [
    ("fp32", 3, 2, 4096),     # 12 items of 12 aimed at
    ("fp32", 3, 3, 2048),     # 12 of 18: halved once
    ("fp32", 3, 4, 2048),     # 24 of 24
    ("fp32", 3, 5, 1024),     # 24 of 30
    ("fp32", 1, 1024, 512),   # 32 of 6144: the smallest chunk
    ("fp64", 1, 5, 512),      # 32 of 30
    ("fp64", 1, 6, 256),      # 32 of 36
    ("fp64", 1, 1024, 128),
])
def test_chunk_follows_items(prec, groups, blocks, chunk):
    assert torch.cuda.is_available()
    D = _segments(N, 1)
    nq = 64 * groups - 63     # a last group of one query segment
    Q = _segments(nq, 2)
    idx = tds.Index(D, num_bins=1)
    got = tds.sort_records(idx.search(Q, 4.0, precision=prec, grid_waves=4 * blocks))
    items = dict(idx.last_stats)["work_items"]
    assert items == groups * (N // chunk)
    want = oracle.sort_results(oracle.search(Q, D, 4.0, -np.inf, np.inf))
    assert want.size > 0
    for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
        assert np.array_equal(got[f], want[f]), f
    # an explicit chunk stays as it is
    idx.search(Q, 4.0, precision=prec, grid_waves=4 * blocks, chunk=8192)
    assert dict(idx.last_stats)["work_items"] == groups * (N // 8192)
    idx.close()
