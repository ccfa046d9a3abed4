"""FP64 plans for several charge vectors: every padded vector count (2, 4, 8, 16 and a
second pass), degrees around the grid lines per row of 16 lanes (n + 1 = 2, 3, 4, 5, 8,
9, 16, and 17 points, which takes the matrix cores), leaves that end inside a block of
16 sources; potentials and modified charges against the oracle (FP64 bar)."""
import numpy as np
import pytest

import oracle
from paper_2003_01836_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    bltc.version()
    return torch.device("cuda:0")


def _soa(pos, dev):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(pos, dtype=np.float64).T)).to(dev)


# vectors, degree, leaf, particles
SHAPES = [(2, 1, 17, 1500), (3, 2, 40, 3000), (4, 3, 80, 5000), (5, 4, 150, 9000), (8, 7, 600, 12000),
          (9, 8, 800, 20000), (16, 8, 1000, 30000), (17, 5, 300, 6000), (20, 3, 70, 2500),
          (3, 15, 4100, 30000), (3, 16, 5000, 30000), (16, 16, 5000, 30000)]


@pytest.mark.parametrize("m,degree,leaf,n", SHAPES)
@pytest.mark.parametrize("kernel,okern,kw,par", [("coulomb", oracle.COULOMB, {}, 0.0),
                                                 ("yukawa", oracle.YUKAWA, {"kappa": 0.5}, 0.5),
                                                 ("regularized", oracle.REGULARIZED, {"delta": 0.01},
                                                  0.01)])
def test_vector_counts(dev, m, degree, leaf, n, kernel, okern, kw, par):
    import paper_2003_01836_amd as bltc
    pos, q = inputs.uniform_cube(n, 985 + degree, m=m)
    t = _soa(pos, dev)
    plan = bltc.Plan(t, t, theta=0.8, degree=degree, leaf_size=leaf, batch_size=leaf, max_q=m,
                     kernel=kernel, **kw)
    got = plan.execute(torch.from_numpy(q).to(dev)).cpu().numpy()
    smp = inputs.sample_indices(n, 500, 986)
    tc = oracle.Treecode(pos, pos, 0.8, degree, leaf, leaf)
    vec = sorted({0, m // 2, m - 1})
    ref = tc.potential(q[vec], kernel=okern, kappa=par, sample=smp)
    for i, v in enumerate(vec):
        assert np.max(np.abs(ref[i] - got[v][smp])) <= 1e-12 * np.max(np.abs(ref[i])), (v,)
    if kernel != "coulomb":
        return
    # modified charges of the last pass, whatever its row length
    view = plan.view()
    used = np.unique(view["item_cluster"][view["item_kind"] == 0])
    one = bltc.Plan(t, t, theta=0.8, degree=degree, leaf_size=leaf, batch_size=leaf, symmetry=False)
    one.execute(torch.from_numpy(q[m - 1]).to(dev))
    for c in used[[0, -1]] if used.size else []:
        a, b = plan.modified_charges(c, qi=m - 1), one.modified_charges(c)
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
