"""Merges that the one-pass form gives up (a pair of more records than its tiles
hold, a record that is no interval): what the general form returns is all that
is seen of them, in the output past the result as well."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from test_emulated_kernels import RESULT_DTYPE, _build_harness


def _records(kind):
    n = 900
    r = np.zeros(n, RESULT_DTYPE)
    r["q_seg"] = np.arange(n)
    r["t_lo"] = 10.0 * np.arange(n)
    r["t_hi"] = r["t_lo"] + 1
    if kind == "long":  # 899 intervals apart, and the last record spans them all
        r["t_lo"][-1], r["t_hi"][-1] = -1.0, 10.0 * n
    else:  # pairs of three, one record in each pair no interval
        r["e_traj"] = np.arange(n) // 3
        r["t_lo"][::3] += 40.0
    return r


def _check(kind, st, m, raw, cap):
    want = oracle.merge_trajectories(_records(kind))
    assert 0 < want.size < cap
    if kind == "long":
        assert want.size == 1
    assert (st, m) == (0, want.size)
    assert raw[:24 * m] == want.tobytes()
    assert raw[24 * m:] == b"\xab" * (24 * (cap - m))


def test_nothing_past_the_result_emulated(tmp_path):
    harness = str(tmp_path / "harness")
    _build_harness(harness)
    recs, out = str(tmp_path / "recs.bin"), str(tmp_path / "out.bin")
    _records("long").tofile(recs)
    r = subprocess.run([harness, "mergefull", recs, "1000", out], capture_output=True, text=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"), timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    st, m = (int(v) for v in r.stdout.split())
    _check("long", st, m, open(out, "rb").read(), 1000)


@pytest.mark.gpu
def test_lengths_of_the_walk():
    """Runs of every length around the eight records that the general form's walk
    reads ahead, behind a run that makes it the form taken."""
    import paper_1410_2698_amd as tds
    rng = np.random.default_rng(3)
    runs = np.concatenate([[1600], np.arange(1, 35).repeat(3)])
    pair = np.repeat(np.arange(runs.size), runs)
    r = np.zeros(pair.size, RESULT_DTYPE)
    r["q_traj"], r["e_traj"] = pair // 9, pair % 9
    r["t_lo"] = rng.integers(0, 160, pair.size) / 4.0
    r["t_hi"] = r["t_lo"] + rng.integers(0, 6, pair.size) / 4.0
    r = r[rng.permutation(r.size)]
    want = oracle.merge_trajectories(r)
    got = tds.merge_trajectories(r)
    assert got.tobytes() == want.tobytes()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["long", "odd"])
def test_nothing_past_the_result_gpu(kind):
    import torch
    import paper_1410_2698_amd as tds
    recs = torch.from_numpy(_records(kind).view(np.uint8).copy()).cuda()
    out = torch.full((1000 * 24,), 0xAB, dtype=torch.uint8, device="cuda")
    st, m = tds.merge_trajectories_raw(recs.data_ptr(), 900, True, out.data_ptr(), 1000, True)
    _check(kind, st, m, out.cpu().numpy().tobytes(), 1000)
