"""The one-pass merge at its tiles' ends, in the form that large inputs take
(tiles of 1,024, keys of 32 and 64 bits, from 2^20 records on) and around the size
at which the tiles grow (2^18): ragged runs of up to 512 records, most of which
straddle a tile's end, in random order, against the oracle."""
import numpy as np
import pytest

import oracle
from test_emulated_kernels import same_intervals
from test_merge_forms import records

pytestmark = pytest.mark.gpu

SMALL = 1 << 18


def _runs(n, low, high, seed):
    """Runs of low..high records, n in all."""
    rng = np.random.default_rng(seed)
    r = rng.integers(low, high + 1, n // low + 1)
    r = r[:np.searchsorted(np.cumsum(r), n)]
    rest = n - int(r.sum())
    return np.append(r, rest) if rest else r


@pytest.mark.parametrize("ids", [1, 60000], ids=["narrow", "wide"])
@pytest.mark.parametrize("low,high,n", [(1, 40, (1 << 20) + 4001), (400, 512, 1 << 20), (511, 512, (1 << 20) + 1)])
def test_large(ids, low, high, n):
    import paper_1410_2698_amd as tds
    recs = records(_runs(n, low, high, n + low), 3, ids=ids)
    assert recs.size == n >= 1 << 20
    same_intervals(tds.merge_trajectories(recs), oracle.merge_trajectories(recs))


@pytest.mark.parametrize("n", [255, 256, 257, 768, 769, 1024, SMALL - 1, SMALL, SMALL + 1])
@pytest.mark.parametrize("low,high", [(1, 90), (200, 512)])
def test_around_the_small_tiles(n, low, high):
    import paper_1410_2698_amd as tds
    recs = records(_runs(n, low, high, n), 4)
    assert recs.size == n
    same_intervals(tds.merge_trajectories(recs), oracle.merge_trajectories(recs))
