"""Mutual leaf pairs planned on the device against the host's plan (which a
workspace limit selects): the same pairs, the same potentials up to the order of
FP64 additions, at leaves of one point, of a multiple of a sub-unit's 512 targets
and one more, with duplicated points, and without any pair."""
import numpy as np
import pytest

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


def _grid(n, side, per):
    """`per` points in each cell of a side^3 grid: leaves of exactly `per` points."""
    g = np.random.default_rng(n)
    cells = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    return ((cells + 0.1 + 0.8 * g.random((side ** 3, per, 3))) / side).reshape(-1, 3)


def _points(case):
    if case == "single":
        return inputs.uniform_cube(300, 990)[0], 1
    if case == "full":
        return _grid(1, 2, 512), 512
    if case == "one over":
        return _grid(2, 2, 513), 513
    if case == "two full":
        return _grid(3, 2, 1024), 1024
    if case == "duplicates":
        pos = inputs.uniform_cube(3000, 991)[0]
        pos[1::3] = pos[::3]
        return pos, 60
    if case == "ragged":
        return inputs.plummer_sphere(20011, 992)[0], 150
    return inputs.uniform_cube(40, 993)[0], 100   # one leaf: no pair


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("method", ["bltc", "cc", "cp"])
@pytest.mark.parametrize("case", ["single", "full", "one over", "two full", "duplicates", "ragged",
                                  "one leaf"])
def test_device_and_host_pair_plans(dev, case, method, precision):
    import paper_2003_01836_amd as bltc
    pos, leaf = _points(case)
    n = pos.shape[0]
    t = torch.from_numpy(np.ascontiguousarray(pos.T)).to(dev)
    q = torch.from_numpy(np.random.default_rng(994).uniform(-1, 1, n)).to(dev)
    kw = dict(theta=0.6, degree=2, leaf_size=leaf, batch_size=leaf, method=method,
              precision=precision)
    device = bltc.Plan(t, t, **kw)
    host = bltc.Plan(t, t, workspace_limit=1 << 40, **kw)
    a, b = device.execute(q).cpu().numpy(), host.execute(q).cpu().numpy()
    sa, sb = device.stats(), host.stats()
    for k in ("mutual_pairs", "mutual_pair_evals", "pair_workspace_bytes", "workspace_bytes",
              "pair_rounds"):
        assert sa[k] == sb[k], k
    assert (sa["mutual_pairs"] > 0) == (case != "one leaf")
    assert np.max(np.abs(a - b)) <= 1e-13 * np.max(np.abs(b))
