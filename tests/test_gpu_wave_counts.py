"""Interaction launches of 1, 2 and 4 waves a workgroup, which take more targets than
the shapes of the other tests: many targets and few sources, on sampled targets against
the oracle's treecode (FP64 bar 1e-12 of the largest potential; FP32-mixed as there).
The wave counts themselves are asserted from the plan's batches."""
import ctypes

import numpy as np
import pytest

import oracle
from tests.conftest import assert_mixed
from paper_2003_01836_amd import _capi, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NS = 3000


@pytest.fixture(scope="module")
def data():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    src, q = inputs.uniform_cube(NS, 1040, m=9)
    s = torch.from_numpy(np.ascontiguousarray(src.T)).to(dev)
    out = {"src": src, "q": q, "s": s, "qd": torch.from_numpy(q).to(dev)}
    for nt in (600000, 2200000):
        tgt, _ = inputs.uniform_cube(nt, 1041)
        out[nt] = (tgt, torch.from_numpy(np.ascontiguousarray(tgt.T)).to(dev),
                   inputs.sample_indices(nt, 1500, 1042))
    return out


def _waves(plan, asked, most, early):
    count = np.asarray(plan.view()["batch_count"])
    groups = int(np.sum((count + 63) // 64))
    f = _capi.load().bltc_internal_waves
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32]
    f.restype = ctypes.c_int32
    return f(int(np.sum(count)), groups, asked, most, early), groups


def _reference(data, nt, leaf, batch, degree, hermite, vec):
    tgt, _, smp = data[nt]
    tc = oracle.Treecode(tgt, data["src"], 0.8, degree, leaf, batch, hermite=hermite)
    return tc.potential(data["q"][vec], sample=smp)


# method, precision, degree, targets, most waves without lanes asked for, early, waves at 1, 2, 4 lanes
ONE = [("bltc", "fp64", 2, 2200000, 16, 1, [1, 2, 4]), ("bltc", "fp32_mixed", 2, 2200000, 16, 0, [1, 2, 4]),
       ("bltc", "fp32_mixed", 11, 2200000, 16, 0, [1, 2, 4]),
       ("bltc", "fp64", 3, 600000, 16, 1, [4, 4, 4]), ("bltc", "fp32_mixed", 3, 600000, 16, 0, [4, 4, 4]),
       ("hermite", "fp64", 2, 2200000, 8, 1, [1, 2, 4]), ("hermite", "fp32_mixed", 4, 2200000, 8, 1, [1, 2, 4]),
       # charges through the scalar cache: no lists shared from 8000 groups on
       ("hermite", "fp32_mixed", 2, 600000, 1, 1, [1, 2, 4])]


@pytest.mark.parametrize("method,precision,degree,nt,most,early,want", ONE)
def test_one_vector(data, method, precision, degree, nt, most, early, want):
    import paper_2003_01836_amd as bltc
    tgt, t, smp = data[nt]
    kw = dict(theta=0.8, degree=degree, leaf_size=100, batch_size=2000, method=method,
              precision=precision)
    ref = _reference(data, nt, 100, 2000, degree, method == "hermite", 0)
    first = None
    for asked, waves in zip((1, 2, 4), want):
        plan = bltc.Plan(t, data["s"], threads_per_target=asked, **kw)
        got = plan.execute(data["qd"][0]).cpu().numpy()
        w, groups = _waves(plan, asked, max(most, asked), early)
        assert w == waves and (most > 1 or groups >= 8000)
        if precision == "fp64":
            assert np.max(np.abs(ref - got[smp])) <= 1e-12 * np.max(np.abs(ref))
        else:
            assert_mixed(ref, got[smp], tgt, data["src"], data["q"][0], idx=smp, what=f"{method} {waves}")
        # the same sums but for the order of FP64 additions
        first = got if first is None else first
        assert np.max(np.abs(got - first)) <= 1e-12 * np.max(np.abs(first))
        plan.close()


# the vector units (2, 3, 5 vectors, FP64), the matrix cores (9 vectors; FP32-mixed)
@pytest.mark.parametrize("nt,waves", [(600000, 4), (2200000, 1)])
@pytest.mark.parametrize("precision,m", [("fp64", 2), ("fp64", 3), ("fp64", 5), ("fp64", 9),
                                         ("fp32_mixed", 3)])
def test_several_vectors(data, precision, m, nt, waves):
    import paper_2003_01836_amd as bltc
    tgt, t, smp = data[nt]
    plan = bltc.Plan(t, data["s"], max_q=m, theta=0.8, degree=3, leaf_size=100, batch_size=2000,
                     precision=precision)
    got = plan.execute(data["qd"][:m].contiguous())[:, torch.from_numpy(smp).to(t.device)].cpu().numpy()
    assert _waves(plan, 1, 8, 0)[0] == waves
    plan.close()
    for v in (0, m - 1):
        ref = _reference(data, nt, 100, 2000, 3, False, v)
        if precision == "fp64":
            assert np.max(np.abs(ref - got[v])) <= 1e-12 * np.max(np.abs(ref))
        else:
            assert_mixed(ref, got[v], tgt, data["src"], data["q"][v], idx=smp, what=f"vector {v}")
