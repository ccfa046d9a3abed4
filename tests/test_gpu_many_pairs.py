"""More mutual leaf pairs than one launch takes: 2^26 units of 64 threads are the 2^32
threads that a grid may not reach.  12,000 points, a leaf each, all pairs direct,
against the oracle's direct sum (FP64 bar: 1e-12 of the largest potential)."""
import numpy as np
import pytest

import oracle
from tests.conftest import assert_mixed
from paper_2003_01836_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_pairs_beyond_2_26(precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    n = 12000
    pos, q = inputs.uniform_cube(n, 1070)
    t = torch.from_numpy(np.ascontiguousarray(pos.T)).to("cuda:0")
    plan = bltc.Plan(t, t, theta=0.0, degree=1, leaf_size=1, batch_size=1, precision=precision)
    st = plan.stats()
    assert st["mutual_pairs"] == n * (n - 1) // 2 > 2 ** 26 and st["pair_rounds"] == 1
    got = plan.execute(torch.from_numpy(q[0]).to("cuda:0")).cpu().numpy()
    plan.close()
    ref = oracle.direct(pos, pos, q[0])
    if precision == "fp64":
        assert np.max(np.abs(ref - got)) <= 1e-12 * np.max(np.abs(ref))
    else:
        assert_mixed(ref, got, pos, pos, q[0], what="pairs")
