"""Pairs whose speed differs by more than FP32's range of squares: the FP32 form
finds what the FP64 form finds, wherever its refinement runs.  The refinement
alone runs on the CPU over a range of speeds, durations and positions."""
import subprocess

import numpy as np
import pytest

import oracle
import trajgen
from test_emulated_kernels import _build_harness


def test_refinement_keeps_every_accepted_pair(tmp_path):
    harness = str(tmp_path / "harness")
    _build_harness(harness)
    r = subprocess.run([harness, "fastpairs", "3", "1000000"], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    st, accepted, misses, past, dropped = (int(v) for v in r.stdout.split())
    assert st == 0
    assert accepted > 100000 and past > 1000 and dropped > 10000
    assert misses == 0


def _pairs(speed, dt, at, n=96):
    """Entry i and query segment i meet head-on in the middle of their common
    extent, near x = i * at."""
    rng = np.random.default_rng(4)
    x = np.arange(n) * at
    t0 = rng.uniform(0, 10, n)

    def seg(sign, off):
        a = np.zeros((8, n))
        a[3], a[7] = t0 + off * dt, t0 + off * dt + dt
        mid = t0 + 0.6 * dt
        a[0], a[4] = x + sign * speed * (a[3] - mid), x + sign * speed * (a[7] - mid)
        a[1] = a[5] = rng.uniform(-1, 1, n) * 0.2 * speed * dt * 1e-3
        return trajgen.Segments(*a, traj=np.arange(n, dtype=np.uint32))
    return seg(1.0, 0.0), seg(-1.0, 0.2), speed * dt * 1e-3


@pytest.mark.gpu
@pytest.mark.parametrize("speed,dt,at", [(1e15, 1e-2, 1e14), (3e18, 1e-2, 1e16), (9e18, 1e-3, 1e15),
                                         (1.2e19, 1e-2, 1e16), (2e19, 1e-3, 1e16), (1e22, 1e-5, 1e15)])
@pytest.mark.parametrize("refine", ["inline", "queued"])
def test_fp32_form_finds_them(speed, dt, at, refine):
    import paper_1410_2698_amd as tds
    D, Q, d = _pairs(speed, dt, at)
    want = oracle.sort_results(oracle.search(Q, D, d, -np.inf, np.inf))
    assert want.size >= len(D)
    idx = tds.Index(D)
    for kw in (dict(precision="fp64"), dict(refine=refine), dict(refine=refine, tile=4)):
        got = tds.sort_records(idx.search(Q, d, **kw))
        assert got.size == want.size, kw
        for f in ("q_seg", "e_seg", "q_traj", "e_traj", "t_lo", "t_hi"):
            assert np.array_equal(got[f], want[f]), (kw, f)
    idx.close()
