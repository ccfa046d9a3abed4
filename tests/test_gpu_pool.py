"""Plans created and destroyed one after the other, on several streams and threads,
their device memory reused without a wait by the caller: each evaluation against the
oracle's treecode (FP64 bar: 1e-12 of the largest potential)."""
import threading

import numpy as np
import pytest

import oracle
from paper_2003_01836_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [(20011, 300), (1, 10), (3001, 60), (19000, 300), (70001, 500), (3001, 60), (257, 16)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    bltc.version()
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def cases(dev):
    out = []
    for k, (n, leaf) in enumerate(SIZES):
        pos, q = inputs.uniform_cube(n, 970 + k)
        ref = oracle.Treecode(pos, pos, 0.7, 3, leaf, leaf).potential(q[0])
        out.append((torch.from_numpy(np.ascontiguousarray(pos.T)).to(dev),
                    torch.from_numpy(q[0]).to(dev), leaf, ref))
    torch.cuda.synchronize()
    return out


def _run(dev, cases, order, rounds):
    """Potentials of every case, plans destroyed while their streams are busy."""
    import paper_2003_01836_amd as bltc
    streams = [torch.cuda.Stream(dev) for _ in range(2)]
    got = []
    for k in range(rounds * len(order)):
        t, q, leaf, _ = cases[order[k % len(order)]]
        with torch.cuda.stream(streams[k % 2]):
            plan = bltc.Plan(t, t, theta=0.7, degree=3, leaf_size=leaf, batch_size=leaf)
            got.append((order[k % len(order)], plan.execute(q)))
        del plan
    for s in streams:
        s.synchronize()
    return got


def _check(cases, got):
    for k, phi in got:
        ref = np.ravel(cases[k][3])
        err = np.max(np.abs(phi.cpu().numpy().ravel() - ref))
        assert err <= 1e-12 * max(np.max(np.abs(ref)), 1e-300), (k, err)


def test_plans_in_turn(dev, cases):
    _check(cases, _run(dev, cases, list(range(len(SIZES))), 3))


def test_plans_of_several_threads(dev, cases):
    results = [None] * 3

    def work(i):
        order = list(range(len(SIZES)))
        results[i] = _run(dev, cases, order[i:] + order[:i], 2)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(results))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for got in results:
        assert got is not None
        _check(cases, got)
