"""The radix sort on either side of the sizes from which its tiles grow (2^18 and
2^23 pairs): index builds (64-bit keys) against numpy's stable order, merges with
32-bit and 64-bit keys, and the merge's general form, against a merge in numpy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu

MEDIUM, LARGE = 1 << 18, 1 << 23


@pytest.mark.parametrize("n", [MEDIUM - 1, MEDIUM, MEDIUM + 1, LARGE - 1, LARGE, LARGE + 1,
                               LARGE + 1024 * 16 * 3 + 777])
@pytest.mark.parametrize("layout", ["temporal", "spatial"])
def test_index_order(n, layout):
    assert torch.cuda.is_available()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    u = torch.rand(7, n, generator=g, device="cuda", dtype=torch.float64)
    ts = (u[6] * 3000).floor() / 8  # many ties
    D = {k: u[i].contiguous() for i, k in enumerate(("xs", "ys", "zs", "xe", "ye", "ze"))}
    D.update(ts=ts.contiguous(), te=(ts + 1).contiguous(), traj=torch.arange(n, dtype=torch.int32, device="cuda"))
    with tds.Index(D, num_bins=5, layout=layout) as idx:
        got = idx.export()
        t_min, width = idx.info()["t_min"], idx.info()["bin_width"]
    ts = ts.cpu().numpy()
    order = got["order"]
    if layout == "temporal":
        assert np.array_equal(order, np.argsort(ts, kind="stable"))
        return
    # by bin; inside a bin a permutation of its entries
    b = np.clip(np.floor((ts - t_min) / width), 0, 4)
    assert np.all(np.diff(b[order]) >= 0)
    assert np.array_equal(np.sort(order), np.arange(n))


def _records(n, pairs, ids, seed, long_run=0):
    """n records of `pairs` trajectory pairs on the GPU, (n, 4) int64; a run of
    long_run records of one more pair if asked."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pair = torch.randint(0, pairs, (n,), generator=g, device="cuda")
    if long_run:
        pair[torch.randperm(n, generator=g, device="cuda")[:long_run]] = pairs
    q, e = (pair // 1000) * ids, (pair % 1000) * ids + 5
    lo = torch.randint(0, 4000, (n,), generator=g, device="cuda").double() / 4
    hi = lo + torch.randint(0, 3, (n,), generator=g, device="cuda").double() / 4
    w = torch.stack([torch.zeros_like(pair), (e << 32) | q, lo.view(torch.int64), hi.view(torch.int64)], 1)
    return w.contiguous(), pair, lo, hi


def _merged(pair, lo, hi):
    """(pair, t_lo, t_hi) of the maximal intervals, by pair and t_lo."""
    pair, lo, hi = (x.cpu().numpy() for x in (pair, lo, hi))
    o = np.lexsort((lo, pair))
    pair, lo, hi = pair[o], lo[o], hi[o]
    first = np.r_[True, pair[1:] != pair[:-1]]
    # running end within a pair: pairs lifted past one another's times
    lift = 1e4 * pair
    reach = np.maximum.accumulate(hi + lift)
    head = first | np.r_[True, (lo + lift)[1:] > reach[:-1]]
    last = np.r_[head[1:], True]
    return pair[head], lo[head], (reach - lift)[last]


@pytest.mark.parametrize("kind", ["narrow", "wide", "general"])
@pytest.mark.parametrize("n", [MEDIUM + 1, (1 << 20) + 5, LARGE - 1, LARGE, LARGE + 1, LARGE + 1024 * 16 * 3 + 777])
def test_merge(n, kind):
    pairs = n // 20  # runs of about 20, across every tile's end
    w, pair, lo, hi = _records(n, pairs, 1 if kind == "narrow" else 100000, n % 1000,
                               1600 if kind == "general" else 0)
    out = torch.empty(n, 3, dtype=torch.int64, device="cuda")
    st, m = tds.merge_trajectories_raw(w.data_ptr(), n, True, out.data_ptr(), n, True)
    p, a, b = _merged(pair, lo, hi)
    assert st == tds.TDS_OK and m == p.size
    ids = 1 if kind == "narrow" else 100000
    raw = out[:m].cpu().numpy()
    got = raw.view(np.uint8).reshape(m, 24).view(tds.TRAJ_DTYPE).reshape(-1)
    assert np.array_equal(got["q_traj"], (p // 1000) * ids)
    assert np.array_equal(got["e_traj"], (p % 1000) * ids + 5)
    assert np.array_equal(got["t_lo"], a)
    assert np.array_equal(got["t_hi"], b)
