"""Grid search at the edges of its batches: one query segment and the sizes
around a workgroup's, query boxes of one cell and of more rows of cells than a
step takes (64), more results than a workgroup keeps (128), batches of one and
of more query segments (from 16384 on)."""
import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu


def _segments(n, seed, span):
    rng = np.random.default_rng(seed)
    a = np.empty((8, n))
    a[0:3] = rng.uniform(0, 40, (3, n))
    a[4:7] = a[0:3] + rng.uniform(-2, 2, (3, n))
    a[3] = rng.uniform(0, 10, n)
    a[7] = a[3] + span
    return trajgen.Segments(*a, traj=np.arange(n, dtype=np.uint32) // 3)


@pytest.mark.parametrize("layout", ["temporal", "spatial"])
@pytest.mark.parametrize("nq,d,cells", [(1, 3.0, 1), (3, 0.5, 9), (4, 60.0, 9), (65, 12.0, 16),
                                        (1000, 2.0, 12), (16383, 1.5, 10), (16384, 1.5, 10),
                                        (40961, 1.0, 10)])
def test_grid_batches(nq, d, cells, layout):
    assert torch.cuda.is_available()
    D, Q = _segments(1500, 5, 0.7), _segments(nq, 6, 0.9)
    idx = tds.Index(D, num_bins=12, layout=layout)
    grid = tds.FSG(idx, cells, cells, cells)
    got = tds.sort_records(grid.search(Q, d))
    want = oracle.sort_results(oracle.search(Q, D, d, -np.inf, np.inf))
    assert got.size == want.size
    for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
        assert np.array_equal(got[f], want[f]), f
    grid.close()
    idx.close()
