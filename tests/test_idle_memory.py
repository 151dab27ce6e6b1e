"""Device memory that closed indexes leave to later ones: given back when asked
for, and safe with several threads that build, search and close at once."""
import threading

import numpy as np
import pytest

import oracle
import trajgen

torch = pytest.importorskip("torch")
import paper_1410_2698_amd as tds  # noqa: E402

pytestmark = pytest.mark.gpu


def _segments(n, seed):
    rng = np.random.default_rng(seed)
    a = np.empty((8, n))
    a[0:3] = rng.uniform(0, 30, (3, n))
    a[4:7] = a[0:3] + rng.uniform(-2, 2, (3, n))
    a[3] = rng.uniform(0, 10, n)
    a[7] = a[3] + 0.8
    return trajgen.Segments(*a, traj=np.arange(n, dtype=np.uint32) // 3)


def test_release_idle_memory():
    assert torch.cuda.is_available()
    tds.release_idle_memory()
    idx = tds.Index(_segments(300000, 1))
    idx.search(_segments(50, 2), 1.0)
    before, held = torch.cuda.mem_get_info()[0], tds.release_idle_memory()
    assert held > 0  # what the build alone needed
    assert torch.cuda.mem_get_info()[0] - before >= held
    idx.close()
    before, held = torch.cuda.mem_get_info()[0], tds.release_idle_memory()
    assert held > 300000 * 120 and held <= 1 << 30
    assert torch.cuda.mem_get_info()[0] - before >= held
    assert tds.release_idle_memory() == 0


def test_threads_build_and_close():
    Q = _segments(100, 3)
    data = [_segments(n, 4 + i) for i, n in enumerate((3000, 40000, 64, 25000))]
    want = [oracle.sort_results(oracle.search(Q, D, 2.0, -np.inf, np.inf)) for D in data]
    wrong = []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for k in range(12):
                    i = (t + k) % len(data)
                    idx = tds.Index(data[i], layout=("spatial", "temporal")[k % 2])
                    got = tds.sort_records(idx.search(Q, 2.0))
                    idx.close()
                    if k % 5 == t:
                        tds.release_idle_memory()
                    if got.tobytes() != want[i].tobytes():
                        wrong.append((t, k))
        except Exception as e:  # reported by the test's thread
            wrong.append((t, repr(e)))
    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
