"""Mutual leaf pairs planned on the device where every leaf sees every other directly:
the lists are as long as there are leaves.  The potentials equal those of the plain
lists up to the order of FP64 additions, and the setup grows with the entries (four
times as many at twice the leaves), not with entries times list length."""
import time

import numpy as np
import pytest

from paper_2003_01836_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KW = dict(theta=0.001, degree=1, leaf_size=1, batch_size=1)


def _points(n):
    pos, q = inputs.uniform_cube(n, 1030)
    return (torch.from_numpy(np.ascontiguousarray(pos.T)).to("cuda:0"),
            torch.from_numpy(q[0]).to("cuda:0"))


@pytest.fixture(scope="module")
def bltc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd
    return paper_2003_01836_amd


@pytest.mark.parametrize("method", ["bltc", "cp", "cc"])
def test_pairs_of_long_lists(bltc, method):
    n = 1500
    t, q = _points(n)
    plan = bltc.Plan(t, t, method=method, **KW)
    assert plan.stats()["mutual_pairs"] == n * (n - 1) // 2
    a = plan.execute(q).cpu().numpy()
    b = bltc.Plan(t, t, method=method, symmetry=False, **KW).execute(q).cpu().numpy()
    assert np.max(np.abs(a - b)) <= 1e-13 * np.max(np.abs(b))


def _setup_seconds(bltc, n):
    t, _ = _points(n)
    best = np.inf
    for _ in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        bltc.Plan(t, t, **KW).close()
        best = min(best, time.perf_counter() - t0)
    return best


def test_setup_grows_with_the_entries(bltc):
    # searching the lists from the front: 10 times (2.5 s); by bisection: 4 (0.74 s)
    assert _setup_seconds(bltc, 8000) <= 6.5 * _setup_seconds(bltc, 4000)
