"""The tuner times what the plan will run: passes of the plan's own number of charge
vectors, and 2 and 4 lanes per target only where they change the launch."""
import statistics

import numpy as np
import pytest

from paper_2003_01836_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _soa(n, seed, dev):
    return torch.from_numpy(np.ascontiguousarray(inputs.uniform_cube(n, seed)[0].T)).to(dev)


def _lines(path):
    out = {}
    for line in path.read_text().splitlines():
        key, value = line.rsplit("|", 1)
        leaf, ms, lanes = value.split()
        out[key] = (int(leaf), float(ms), int(lanes))
    return out


def _milliseconds(plan, q):
    out = torch.empty((q.shape[0], plan.nt), dtype=torch.float64, device=q.device)
    times = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        plan.execute(q, out=out)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return statistics.median(times)


def test_several_vectors_are_timed_as_they_run(dev, tmp_path, monkeypatch):
    import paper_2003_01836_amd as bltc
    t = _soa(100000, 1050, dev)
    kw = dict(theta=0.7, degree=6)
    for m, padded in ((3, 4), (16, 16)):
        ratios = []
        for attempt in range(3):   # one timing each: the least disturbed counts
            cache = tmp_path / f"tune{m}-{attempt}.txt"
            monkeypatch.setenv("BLTC_TUNE_CACHE", str(cache))
            plan = bltc.Plan(t, t, max_q=m, leaf_size=0, batch_size=0, **kw)
            (key, (leaf, ms, lanes)), = _lines(cache).items()
            assert key.startswith("v3 ") and f" q={padded} " in key and lanes == 1
            assert plan.stats()["leaf_size"] == leaf
            q = torch.ones((m, 100000), dtype=torch.float64, device=dev)
            ratios.append(ms / _milliseconds(plan, q))
            plan.close()
        # the recorded time is that of m vectors (16 take twice as long as 3)
        assert 0.6 <= min(ratios) <= 1.4


def test_identical_launches_are_not_compared(dev):
    # 16 waves a workgroup whatever the lanes: one lane is reported
    import paper_2003_01836_amd as bltc
    t = _soa(5000, 1051, dev)
    for method in ("bltc", "hermite"):
        for precision in ("fp64", "fp32_mixed"):
            for _ in range(3):
                leaf, lanes, ms = bltc.autotune(t, t, candidates=(200, 500), use_cache=False, full=True,
                                                theta=0.7, degree=2, method=method,
                                                precision=precision)
                assert lanes == 1 and leaf in (200, 500) and ms > 0


def test_lanes_are_searched_where_they_count(dev):
    # 2.2 10^6 targets: one wave a workgroup unless more lanes are asked for
    import paper_2003_01836_amd as bltc
    t, s = _soa(2200000, 1052, dev), _soa(2000, 1053, dev)
    leaf, lanes, ms = bltc.autotune(t, s, candidates=(1000,), use_cache=False, full=True, theta=0.7,
                                    degree=2)
    assert leaf == 1000 and lanes in (1, 2, 4) and ms > 0
