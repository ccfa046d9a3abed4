"""Idle device memory of destroyed plans: given back on request, and when an
allocation of the library finds the device out of memory."""
import ctypes

import numpy as np
import pytest

from paper_2003_01836_amd import _capi, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _idle_blocks(bltc):
    """Leaves some 200 MB of idle blocks behind; the potentials of the plan."""
    pos, q = inputs.uniform_cube(200000, 1060)
    t = torch.from_numpy(np.ascontiguousarray(pos.T)).to("cuda:0")
    plan = bltc.Plan(t, t, theta=0.7, degree=4, leaf_size=500, batch_size=500)
    phi = plan.execute(torch.from_numpy(q[0]).to("cuda:0"))
    held = plan.stats()["workspace_bytes"]
    plan.close()
    return phi, held


@pytest.fixture(scope="module")
def bltc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd
    first, _ = _idle_blocks(paper_2003_01836_amd)   # modules and torch's own memory
    return paper_2003_01836_amd


def test_release_memory(bltc):
    a, held = _idle_blocks(bltc)
    assert held > 100e6
    before = _free()
    bltc.release_memory()
    assert _free() - before > 0.8 * held
    bltc.release_memory()   # nothing left
    b, _ = _idle_blocks(bltc)
    assert torch.equal(a, b)


def test_out_of_memory_gives_back_idle_blocks(bltc):
    f = _capi.load().bltc_internal_try_alloc
    f.argtypes, f.restype = [ctypes.c_int64], ctypes.c_int
    assert f(1 << 30) == 0
    _, held = _idle_blocks(bltc)
    before = _free()
    assert f(1 << 42) != 0      # 4 TiB: refused, after the idle blocks were freed
    assert _free() - before > 0.8 * held
