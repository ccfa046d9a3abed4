"""Target and source orders of device-built plans: permutations that put the particles
into the batches' boxes, at sizes around the block of records that is read back at a
time, and in a time that a copy of whole records takes many times over."""
import time

import numpy as np
import pytest

from paper_2003_01836_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["bltc", "cp", "cc"])
@pytest.mark.parametrize("n", [1, 16, 2 ** 18, 2 ** 18 + 1, 600000])
def test_orders_of_a_view(n, method):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    dev = torch.device("cuda:0")
    tgt, _ = inputs.uniform_cube(n, 1020)
    src, _ = inputs.uniform_cube(500, 1021)
    t = torch.from_numpy(np.ascontiguousarray(tgt.T)).to(dev)
    s = torch.from_numpy(np.ascontiguousarray(src.T)).to(dev)
    plan = bltc.Plan(t, s, theta=0.7, degree=2, leaf_size=200, batch_size=200, method=method)
    # the device side exists before the clock runs
    plan.execute(torch.ones(500, dtype=torch.float64, device=dev))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    view = plan.view()
    seconds = time.perf_counter() - t0
    order = np.asarray(view["target_order"])
    assert np.array_equal(np.sort(order), np.arange(n))
    assert np.array_equal(np.sort(np.asarray(view["source_order"])), np.arange(500))
    if method == "bltc":
        begin, count = np.asarray(view["batch_begin"]), np.asarray(view["batch_count"])
        lo = np.asarray(view["batch_lo"]).reshape(-1, 3)
        hi = np.asarray(view["batch_hi"]).reshape(-1, 3)
        x = tgt[order]
        for b in {0, begin.size // 2, begin.size - 1}:
            part = x[begin[b]:begin[b] + count[b]]
            assert np.array_equal(part.min(0), lo[b]) and np.array_equal(part.max(0), hi[b])
    # 19 MB of records: some 5 ms; row by row 4 s
    assert seconds < 1.0
