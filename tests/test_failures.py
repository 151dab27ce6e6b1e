"""Calls whose allocations fail, on the CPU: the library's host paths compiled
against the emulation of the kernels, with allocations that fail when told to
(tests/emu/faults.cpp, built with AddressSanitizer)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1410_2698_amd", "csrc")


@pytest.fixture(scope="module")
def faults(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("faults") / "faults")
    cxx = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    cxx = cxx if os.path.exists(cxx) else shutil.which("clang++")
    if cxx is None:
        pytest.skip("clang++ not available")
    emu = os.path.join(ROOT, "tests", "emu")
    src = [os.path.join(CSRC, f + ".hip") for f in ("search", "fsg", "radix_sort", "traj_merge", "index_build",
                                                    "host_search")]
    r = subprocess.run([cxx, "-std=c++20", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer",
                        "-ffp-contract=off", "-Wno-unknown-attributes", "-Wno-ignored-attributes", "-I", emu,
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        "-include", os.path.join(emu, "faults.hpp"), "-x", "c++", *src, "-x", "none",
                        os.path.join(emu, "faults.cpp"), "-o", out, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(*args):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=1")
        r = subprocess.run([out, *args], capture_output=True, text=True, env=env, timeout=600)
        assert r.returncode == 0, (args, r.returncode, r.stderr[-4000:])
        return [int(v) for v in r.stdout.split()]
    return run


@pytest.mark.parametrize("entry", ["search", "batch", "begin"])
def test_failed_call_leaves_no_work_behind(faults, entry):
    """A workspace goes back to its index when a call fails: nothing that was
    queued for it (the query arrays' copy from its pinned memory) may still run."""
    failed, late, unwaited = faults("waits", entry)
    assert failed > 10 and late > 0
    assert unwaited == 0


def test_failed_grid_search_leaves_no_work_behind(faults):
    """The counters go back to the grid's pool when a search fails."""
    failed, late, unwaited = faults("grid")
    assert failed == late == 1
    assert unwaited == 0


def test_failed_merge_leaves_no_work_behind(faults):
    """The merge's scratch is the next merge's, on whatever stream."""
    failed, late, unwaited, counted = faults("merge")
    assert failed > 5 and late > 1
    assert unwaited == 0 and counted == 0


def test_pools_need_no_host_memory(faults):
    """Giving a block back allocates nothing: it happens in destructors and at the
    end of C entries, where an exception ends the program."""
    assert faults("pools") == [0]


def test_searches_without_pinned_memory(faults):
    """The pinned block only saves copies: without one the arrays are copied as
    they are."""
    assert faults("pinned") == [0, 1] * 3


def test_idle_blocks_go_back(faults):
    """Closed indexes leave device blocks to the next; all of them go back when
    asked for, and when an allocation finds no memory."""
    left, freed, left_then, status = faults("trim")
    assert left > 0 and freed >= left << 21
    assert left_then == 0
    assert status == 0
