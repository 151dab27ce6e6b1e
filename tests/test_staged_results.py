"""Staged results that outlast a work item (up to 64 requests) and those that do
not (65): many items per wave, several stages full, slices that hold all of a
request's results, fewer and none."""
import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu

FIELDS = ("xs", "ys", "zs", "ts", "xe", "ye", "ze", "te")


@pytest.fixture(scope="module")
def walks():
    assert torch.cuda.is_available()
    w = trajgen.dense(0.05, n_pts=81)
    idx = tds.Index(w.D)
    want = oracle.search(w.Q, w.D, 12.0, *w.window)
    yield w, idx, want
    idx.close()


def _key(r):
    return r["q_seg"].astype(np.uint64) << np.uint64(32) | r["e_seg"]


@pytest.mark.parametrize("grid_waves", [4, 256])
@pytest.mark.parametrize("nreq", [1, 2, 63, 64, 65])
def test_batches(walks, nreq, grid_waves):
    w, idx, want = walks
    nq = len(w.Q.xs)
    at = np.linspace(0, nq, nreq + 1).astype(int)
    assert want.size > 4 * 4 * 2048  # the stages of 4 waves fill up several times
    parts, reqs, off = [], [], 0
    for i in range(nreq):
        p = want[(want["q_seg"] >= at[i]) & (want["q_seg"] < at[i + 1])].copy()
        p["q_seg"] -= np.uint32(at[i])
        parts.append(oracle.sort_results(p))
        cap = (p.size, p.size + 7, p.size // 2, 0)[i % 4]
        reqs.append((at[i], at[i + 1] - at[i], 12.0, *w.window, off, cap))
        off += cap + 1  # one record between the slices
    out = np.zeros(off, tds.RESULT_DTYPE)
    out["q_seg"] = 0xABABABAB
    st, counts, _ = idx.search_batch_raw(w.Q, reqs, out_ptr=out.ctypes.data, out_capacity=off,
                                         out_on_device=False, grid_waves=grid_waves, output="staged")
    assert counts == [p.size for p in parts]
    assert st == (tds.TDS_OK if nreq < 3 else tds.TDS_E_OVERFLOW)
    for p, r in zip(parts, reqs):
        n = min(p.size, r[6])
        got = tds.sort_records(out[r[5]:r[5] + n])
        assert np.unique(_key(got)).size == n
        same = p[np.searchsorted(_key(p), _key(got))] if n else p[:0]
        for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
            assert np.array_equal(got[f], same[f]), f


@pytest.mark.parametrize("grid_waves", [4, 256])
def test_one_request(walks, grid_waves):
    w, idx, want = walks
    want = oracle.sort_results(want)
    for precision in ("fp32", "fp64"):
        got = tds.sort_records(idx.search(w.Q, 12.0, *w.window, output="staged", precision=precision,
                                          grid_waves=grid_waves, capacity=want.size))
        assert got.tobytes() == want.tobytes()
    # windows of a device buffer that holds a few items' results
    got = tds.sort_records(idx.search(w.Q, 12.0, *w.window, output="staged", capacity=want.size,
                                      device_capacity=want.size // 5, grid_waves=grid_waves))
    assert got.tobytes() == want.tobytes()
