"""The fill of direct output for launches whose waves start with a chunk each
(k_fill), in the CPU emulation of the kernels: reservations of one and more chunks,
untouched first chunks, chunks that are no power of two, capacities of nothing, one,
on a chunk's edge, at, below and past the number of results."""
import concurrent.futures as cf
import os
import subprocess

import numpy as np
import pytest

from test_emulated_kernels import RESULT_DTYPE, _build_harness

# seed, waves, chunk, most chunks of a reservation, results per wave at most,
# capacity = floor(count * frac) + add, rounded down to whole chunks if align
CASES = {
    "exact": (1, 64, 64, 4, 900, 1.0, 0, 0),
    "room": (2, 64, 512, 4, 3000, 1.0, 5000, 0),
    "one_short": (3, 36, 64, 1, 300, 1.0, -1, 0),
    "half": (4, 200, 128, 2, 700, 0.5, 0, 0),
    "edge": (5, 200, 448, 4, 2500, 0.6, 0, 1),
    "odd_chunk": (6, 48, 192, 4, 2500, 0.9, 3, 0),
    "nothing": (7, 16, 64, 4, 400, 0.0, 0, 0),
    "one": (8, 16, 64, 4, 400, 0.0, 1, 0),
    "empty": (9, 16, 512, 4, 0, 1.0, 0, 0),
    "few": (10, 4096, 512, 4, 2, 1.0, 0, 0),
    "most": (11, 4096, 64, 4, 300, 0.8, 0, 0),
    "one_block": (12, 4, 512, 4, 9000, 1.0, 10, 0),
}


@pytest.fixture(scope="module")
def runs(tmp_path_factory):
    base = tmp_path_factory.mktemp("fill")
    harness = str(base / "harness")
    _build_harness(harness)

    def run(name):
        prefix = str(base / name)
        r = subprocess.run([harness, "fillgiven", *map(str, CASES[name]), prefix], capture_output=True,
                           text=True, timeout=900, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=1"))
        return r, prefix
    with cf.ThreadPoolExecutor(4) as ex:
        return dict(zip(CASES, ex.map(run, CASES)))


@pytest.mark.parametrize("name", list(CASES))
def test_fill(runs, name):
    r, prefix = runs[name]
    assert r.returncode == 0, r.stderr[-4000:]
    st, count, cap, T, holes, R, found, tests = (int(v) for v in r.stdout.split())
    waves = CASES[name][1]
    assert st == 0 and T == min(count, cap)
    assert found == count
    assert tests == (waves // 4) * (waves // 4 + 1) // 2
    allr, before, after = (np.fromfile(prefix + x, dtype=RESULT_DTYPE) for x in (".all", ".before", ".after"))
    assert allr.size == count and before.size == after.size == T
    hole = before["q_seg"] == 0xFFFFFFFF
    assert int(hole.sum()) == holes and R >= count + holes
    assert not np.any(after["q_seg"] == 0xFFFFFFFF)
    # records are results as they were placed, each once; those below T stay
    assert np.array_equal(after["e_seg"], allr["e_seg"][after["q_seg"]])
    assert np.unique(after["q_seg"]).size == T
    assert np.array_equal(after[~hole], before[~hole])
    # the holes take the first results past T, all of which were kept
    pos = allr["e_seg"].astype(np.int64)
    assert np.array_equal(np.sort(after["e_seg"][hole].astype(np.int64)), np.sort(pos[pos >= T])[:holes])
    assert np.all(allr["e_traj"][after["q_seg"][hole]] == 1)
    if name in ("exact", "room", "few", "one_block"):
        assert count and np.array_equal(np.sort(after["q_seg"]), np.arange(count))
    if name == "empty":
        assert count == 0
