"""Direct output at the edges of its fill: launches of few waves and of the most
that one fill kernel takes and more, capacities around the number of results.
The records kept are some of the oracle's, each once, as many as fit."""
import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def walks():
    assert torch.cuda.is_available()
    w = trajgen.dense(0.05, n_pts=81)
    idx = tds.Index(w.D)
    want = oracle.sort_results(oracle.search(w.Q, w.D, 12.0, *w.window))
    yield w, idx, want
    idx.close()


@pytest.mark.parametrize("grid_waves", [4, 64, 4096, 4100])
@pytest.mark.parametrize("room", ["none", "one", "third", "less", "all", "more"])
def test_fill_edges(walks, grid_waves, room):
    w, idx, want = walks
    n = want.size
    assert n > 3 * 2048  # several reservations for each of a few waves
    cap = {"none": 0, "one": 1, "third": n // 3, "less": n - 1, "all": n, "more": n + 1000}[room]
    buf = torch.full(((n + 1000) * 32,), 0xAB, dtype=torch.uint8, device="cuda")
    st, m, _ = idx.search_raw(w.Q, 12.0, *w.window, out_ptr=buf.data_ptr(), capacity=cap,
                              out_on_device=True, output="direct", grid_waves=grid_waves)
    assert m == n and st == (tds.TDS_OK if cap >= n else tds.TDS_E_OVERFLOW)
    raw = buf.cpu().numpy()
    k = min(cap, n)
    assert np.all(raw[32 * cap:] == 0xAB)  # within the capacity, the rest is scratch
    got = tds.sort_records(raw[:32 * k].view(want.dtype))
    key = lambda r: r["q_seg"].astype(np.uint64) << np.uint64(32) | r["e_seg"]  # noqa: E731
    assert np.unique(key(got)).size == k
    same = want[np.searchsorted(key(want), key(got))] if k else want[:0]
    for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
        assert np.array_equal(got[f], same[f]), f


@pytest.mark.parametrize("cap", [0, 1, 2047, 2048, 2049, 4096])
@pytest.mark.parametrize("refine", ["default", "queued"])
def test_default_output_by_capacity(walks, cap, refine):
    """Staged up to 32 records per wave (2048 for 64 waves), direct beyond: a
    full output of distinct results and the whole count on either side."""
    w, idx, want = walks
    buf = torch.full(((cap + 64) * 32,), 0xAB, dtype=torch.uint8, device="cuda")
    st, m, _ = idx.search_raw(w.Q, 12.0, *w.window, out_ptr=buf.data_ptr(), capacity=cap,
                              out_on_device=True, grid_waves=64, refine=refine)
    assert m == want.size and st == tds.TDS_E_OVERFLOW
    raw = buf.cpu().numpy()
    assert np.all(raw[32 * cap:] == 0xAB)
    got = tds.sort_records(raw[:32 * cap].view(want.dtype))
    key = lambda r: r["q_seg"].astype(np.uint64) << np.uint64(32) | r["e_seg"]  # noqa: E731
    assert np.unique(key(got)).size == cap
    same = want[np.searchsorted(key(want), key(got))] if cap else want[:0]
    for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
        assert np.array_equal(got[f], same[f]), f
