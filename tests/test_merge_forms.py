"""The trajectory merge where its forms meet: tiles of 1,024 sorted records,
runs that reach past a tile's end, runs of up to 512 records (one pass) and
longer ones (general form), records that are no intervals (general form), and
key widths.  Every result equals the oracle's merge exactly.  Small inputs run
in the CPU emulation of the kernels, all of them on the GPU."""
import concurrent.futures as cf

import numpy as np
import pytest

import oracle
from test_emulated_kernels import RESULT_DTYPE, _build_harness, _run_job, same_intervals


def records(runs, seed, ids=1, quarter=False, odd=0):
    """Records of len(runs) trajectory pairs, runs[i] of them for pair i, in
    random order; times on a grid, so that starts tie and intervals touch."""
    rng = np.random.default_rng(seed)
    pair = np.repeat(np.arange(len(runs)), runs)
    n = pair.size
    r = np.zeros(n, RESULT_DTYPE)
    r["q_seg"] = np.arange(n)
    r["q_traj"] = (pair // 7) * ids
    r["e_traj"] = (pair % 7) * ids + 3
    lo = rng.integers(-4 * 60, 4 * 60, n) / 4.0
    r["t_lo"] = np.where((lo == 0) & (pair % 2 == 1), -0.0, lo)
    r["t_hi"] = lo + rng.integers(0, 6, n) / 4.0
    if odd:  # ends before it starts
        at = rng.choice(n, odd, replace=False)
        r["t_hi"][at] = r["t_lo"][at] - 0.5
    return r[rng.permutation(n)]


SMALL = {
    "one": lambda: records([1], 1),
    "below_tile": lambda: records([1] * 1023, 2),
    "tile": lambda: records([2] * 512, 3),
    "past_tile": lambda: records([5] * 205, 4),
    "run_512": lambda: records([1, 512, 3, 512, 511, 2], 5),
    "run_513": lambda: records([1, 513, 3], 6),
    "run_over_tiles": lambda: records([3, 2500, 1], 7),
    "ragged": lambda: records(np.random.default_rng(8).integers(1, 90, 70), 8, ids=0x10000001),
    "odd": lambda: records([4] * 300, 9, odd=5),
}


@pytest.fixture(scope="module")
def emulated(tmp_path_factory):
    base = tmp_path_factory.mktemp("merge")
    harness = str(base / "harness")
    _build_harness(harness)
    with cf.ThreadPoolExecutor(4) as ex:
        futs = {k: ex.submit(_run_job, harness, str(base / k), "merge", f(), [4000]) for k, f in SMALL.items()}
        return {k: f.result() for k, f in futs.items()}


@pytest.mark.parametrize("name", list(SMALL))
def test_merge_forms_emulated(emulated, name):
    r, out = emulated[name]
    assert r.returncode == 0, r.stderr[-4000:]
    want = oracle.merge_trajectories(SMALL[name]())
    assert [int(v) for v in r.stdout.split()] == [0, want.size]
    same_intervals(np.fromfile(out, dtype=oracle.TRAJ_DTYPE), want)


LARGE = {
    # at and past the size from which the host plans the passes: ids of a few
    # bits (32-bit keys) and of all bits (64-bit keys)
    "narrow": lambda: records(np.random.default_rng(10).integers(1, 40, 52500), 10),
    "wide": lambda: records(np.random.default_rng(11).integers(1, 40, 52500), 11, ids=60000),
    "below": lambda: records([1] * ((1 << 20) - 1), 12),
    "at": lambda: records([2] * (1 << 19), 13),
    "long_run": lambda: records([2] * (1 << 19) + [800], 14),
    "odd_large": lambda: records([2] * (1 << 19), 15, odd=3),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(SMALL) + list(LARGE))
def test_merge_forms_gpu(name):
    import paper_1410_2698_amd as tds
    recs = {**SMALL, **LARGE}[name]()
    want = oracle.merge_trajectories(recs)
    same_intervals(tds.merge_trajectories(recs), want)
    # a capacity below the total keeps the first intervals in order
    cap = max(1, want.size // 3)
    out = np.zeros(cap, oracle.TRAJ_DTYPE)
    st, n = tds.merge_trajectories_raw(recs.ctypes.data, recs.size, False, out.ctypes.data, cap, False)
    assert n == want.size and st == (tds.TDS_OK if n <= cap else tds.TDS_E_OVERFLOW)
    same_intervals(out, want[:cap])
