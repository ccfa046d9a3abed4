"""bltc_direct and bltc_direct_noalloc with the potentials written over the charges:
more potentials than the fixed array holds partial sums for (2^22), and several charge
vectors.  Reference: the same call into memory of its own, whose first targets are held
to the oracle's direct sum (FP64 bar: 1e-12 of the largest potential); the sums run in
the same order, so the potentials are equal bit for bit."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2003_01836_amd import _capi, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    bltc.version()
    return torch.device("cuda:0")


def _call(noalloc, t, s, q, num_q, q_ld, phi, phi_ld):
    """The C entry on raw pointers: rows of charges and potentials at any distance."""
    import paper_2003_01836_amd as bltc
    lib = _capi.load()
    p = bltc.params()
    ptr = [ctypes.c_void_p(r.data_ptr()) for r in (*t, *s, q, phi)]
    fn = lib.bltc_direct_noalloc if noalloc else lib.bltc_direct
    _capi.check(fn(ctypes.byref(p), t.shape[1], *ptr[:3], s.shape[1], *ptr[3:6], ptr[6], num_q, q_ld,
                   ptr[7], phi_ld, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))


# targets, sources, vectors: one piece whose potentials outnumber 2^22 (one and two
# vectors), one that just fits, several pieces with a second pass of vectors
@pytest.mark.parametrize("noalloc", [True, False])
@pytest.mark.parametrize("nt,ns,m", [(2 ** 22 + 65, 3001, 1), (2 ** 21 + 1, 1030, 2), (2 ** 22, 515, 1),
                                     (3001, 3001, 6)])
def test_potentials_over_the_charges(dev, nt, ns, m, noalloc):
    pos, q = inputs.uniform_cube(ns, 1010 + m, m=m)
    tgt, _ = inputs.uniform_cube(nt, 1011 + m)
    t = torch.from_numpy(np.ascontiguousarray(tgt.T)).to(dev)
    s = torch.from_numpy(np.ascontiguousarray(pos.T)).to(dev)
    buf = torch.full((m, nt), np.nan, dtype=torch.float64, device=dev)
    buf[:, :ns] = torch.from_numpy(q).to(dev)
    charges = buf.clone()
    ref = torch.empty_like(buf)
    _call(noalloc, t, s, charges, m, nt, ref, nt)
    _call(noalloc, t, s, buf, m, nt, buf, nt)
    assert torch.equal(buf, ref)
    few = oracle.direct(tgt[:200], pos, q)
    got = ref[:, :200].cpu().numpy()
    assert np.max(np.abs(few - got)) <= 1e-12 * np.max(np.abs(few))
