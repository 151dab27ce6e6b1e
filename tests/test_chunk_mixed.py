"""Candidates per work item (chunk = 0) where times are mixed: entries with start
times of their own, bins wider than a segment, buckets that span bins.  The chunk
is halved once, and then not where that takes the items from at most one per wave
to more; up to there and past it as for others."""
import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu

N = 16384


def _segments(n, seed, wide):
    """Segments of length 1 that begin in [0, 3], or (not wide) all over [0, 1]."""
    rng = np.random.default_rng(seed)
    a = np.empty((8, n))
    a[0:3] = rng.uniform(0, 40, (3, n))
    a[4:7] = a[0:3] + rng.uniform(-1, 1, (3, n))
    a[3] = rng.uniform(0, 3, n) if wide else 0.0
    a[7] = a[3] + 1.0
    return trajgen.Segments(*a, traj=np.arange(n, dtype=np.uint32))


@pytest.mark.parametrize("prec,groups,blocks,wide,chunk", [
    ("fp32", 3, 5, True, 1024),     # 24 items do not fit 20 waves and are short of the 30 aimed at
    ("fp32", 3, 6, True, 2048),     # 24 of 24 waves fit, 48 do not
    ("fp32", 3, 12, True, 1024),    # 48 fit, 96 do not
    ("fp32", 3, 24, True, 512),     # 96 fit
    ("fp32", 3, 24, False, 512),    # times in common: as far as the items aimed at
    ("fp32", 3, 12, False, 512),
    ("fp64", 1, 32, True, 128),     # 128 items of 192 aimed at: fp64 does not ask
])
def test_chunk_of_mixed_times(prec, groups, blocks, wide, chunk):
    assert torch.cuda.is_available()
    D = _segments(N, 1, wide)
    Q = _segments(64 * groups - 63, 2, wide)
    if wide:  # every query begins in the one bin
        assert (D.te.max() - D.ts.min()) > 1.5
    idx = tds.Index(D, num_bins=1)
    got = tds.sort_records(idx.search(Q, 4.0, precision=prec, grid_waves=4 * blocks))
    assert dict(idx.last_stats)["work_items"] == groups * (N // chunk)
    want = oracle.sort_results(oracle.search(Q, D, 4.0, -np.inf, np.inf))
    assert want.size > 0
    for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
        assert np.array_equal(got[f], want[f]), f
    idx.close()
