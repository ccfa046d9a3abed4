"""The direct sum's split of the sources over waves and workgroups, at its edges,
against the oracle's direct sum (FP64 bar: 1e-12 of the largest potential)."""
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


def _check(ref, got):
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(ref - got)) <= 1e-12 * np.max(np.abs(ref))


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("nt,ns,m", [(1, 1, 1), (1, 1027, 2), (63, 3, 4), (64, 255, 3), (65, 257, 5),
                                     (1000, 20003, 1), (129, 70001, 9), (4097, 64, 2)])
def test_direct_split_edges(dev, nt, ns, m, noalloc):
    import paper_2003_01836_amd as bltc
    pos, q = inputs.uniform_cube(ns, 950 + nt, m=m)
    tgt, _ = inputs.uniform_cube(nt, 951 + ns)
    tgt[0] = pos[0]            # a pair at zero distance
    if ns > 1:
        pos[-1] = pos[0]       # ... twice
    for kernel, okern, kw in (("coulomb", oracle.COULOMB, {}), ("yukawa", oracle.YUKAWA, {"kappa": 0.5})):
        got = bltc.direct(_soa(tgt, dev), _soa(pos, dev), torch.from_numpy(q).to(dev), kernel=kernel,
                          noalloc=noalloc, **kw).cpu().numpy()
        ref = oracle.direct(tgt, pos, q, kernel=okern, kappa=kw.get("kappa", 0.0))
        if ns == 1:
            assert np.array_equal(got, np.zeros((m, nt)))
        else:
            _check(ref, got)


@pytest.mark.parametrize("noalloc", [False, True])
def test_direct_potentials_over_the_charges(dev, noalloc):
    # out is the charges' own tensor: every charge is read before a potential is written
    import paper_2003_01836_amd as bltc
    pos, q = inputs.uniform_cube(3001, 960)
    t = _soa(pos, dev)
    qd = torch.from_numpy(q[0]).to(dev)
    got = bltc.direct(t, t, qd, out=qd, noalloc=noalloc)
    assert got.data_ptr() == qd.data_ptr()
    _check(oracle.direct(pos, pos, q[0]), got.cpu().numpy())


@pytest.mark.parametrize("kappa", [1e-3, 0.5, 2.0, 30.0, 1e4])
def test_yukawa_over_its_exponents(dev, kappa):
    # one source: each value against exp(-kappa r^2 g) g with g the Coulomb value 1/r of
    # the same pair (so the reciprocal square root's own error, one Newton step from the
    # hardware's 2^-24, is left out), from exponents near 0 through every table entry
    # to underflow; 16 half ulps of the value and of the exponent allowed
    import paper_2003_01836_amd as bltc
    x = np.concatenate([np.geomspace(1e-6, 800.0, 20011), [1e5, 1e12, 1e60]])   # kappa r
    pos = np.zeros((x.size, 3))
    pos[:, 0] = x / kappa
    src = _soa(np.zeros((1, 3)), dev)
    one = torch.ones(1, dtype=torch.float64, device=dev)
    got = bltc.direct(_soa(pos, dev), src, one, kernel="yukawa", kappa=kappa).cpu().numpy().ravel()
    g = bltc.direct(_soa(pos, dev), src, one).cpu().numpy().ravel().astype(np.longdouble)
    r2 = pos[:, 0].astype(np.longdouble) ** 2
    ref = (np.exp(-np.longdouble(kappa) * r2 * g) * g).astype(np.float64)
    tol = 16.0 * (1.0 + x) * 2.0 ** -53
    assert np.all(np.abs(got - ref) <= tol * ref + 1e-307)
