"""Interaction lists shared by the waves of a workgroup: the numbers of waves that
a launch picks (16, 8, 4 and, with sub-blocks of a 256-target group, 1), list
parts that start inside a cluster's planes or a leaf's 128-source blocks, and
lists longer than the 64 entries a wave scans at once; against the oracle."""
import numpy as np
import pytest

import oracle
from tests.conftest import assert_mixed
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


# targets, sources, degree, leaf, theta
SHAPES = [(1, 3000, 2, 40, 0.5),        # one target, over 64 direct leaves
          (65, 5000, 3, 700, 0.8),      # leaves of several 128-source blocks
          (2000, 4000, 2, 30, 0.4),     # hundreds of small leaves per batch
          (40000, 6000, 2, 100, 0.8),   # 8 waves
          (150000, 2000, 3, 300, 0.8)]  # 4 waves


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("method", ["bltc", "hermite"])
@pytest.mark.parametrize("nt,ns,degree,leaf,theta", SHAPES)
def test_wave_split(dev, nt, ns, degree, leaf, theta, method, precision):
    import paper_2003_01836_amd as bltc
    src, q = inputs.uniform_cube(ns, 970 + degree)
    tgt, _ = inputs.uniform_cube(nt, 971 + nt)
    t, s, qd = _soa(tgt, dev), _soa(src, dev), torch.from_numpy(q[0]).to(dev)
    kw = dict(theta=theta, degree=degree, leaf_size=leaf, batch_size=leaf, method=method,
              precision=precision)
    got = bltc.Plan(t, s, **kw).execute(qd).cpu().numpy()
    smp = inputs.sample_indices(nt, 2000, 972)
    ref = oracle.Treecode(tgt, src, theta, degree, leaf, leaf,
                          hermite=method == "hermite").potential(q[0], sample=smp)
    if precision == "fp64":
        assert np.max(np.abs(ref - got[smp])) <= 1e-12 * np.max(np.abs(ref))
    else:
        assert_mixed(ref, got[smp], tgt, src, q[0], idx=smp, what=f"{method} {nt}")
    # four lanes asked for: the same sums but for the order of FP64 additions
    four = bltc.Plan(t, s, threads_per_target=4, **kw).execute(qd).cpu().numpy()
    assert np.max(np.abs(four - got)) <= 1e-12 * np.max(np.abs(got))


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_wave_split_of_256_target_groups(dev, precision):
    # one charge vector through a plan for several: groups of 256 targets
    import paper_2003_01836_amd as bltc
    pos, q = inputs.uniform_cube(5000, 980, m=2)
    t = _soa(pos, dev)
    qd = torch.from_numpy(q).to(dev)
    kw = dict(theta=0.7, degree=4, leaf_size=333, batch_size=333, precision=precision)
    plan = bltc.Plan(t, t, max_q=2, **kw)
    one = bltc.Plan(t, t, symmetry=False, **kw)
    for m in range(2):
        a = plan.execute(qd[m]).cpu().numpy()
        b = one.execute(qd[m]).cpu().numpy()
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
