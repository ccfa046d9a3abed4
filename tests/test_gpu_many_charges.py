"""Charges of more sources and vectors than one launch gathers (2^28 sources times 16
vectors are the 2^32 threads that a grid may not reach): 1000 targets, all direct,
against the library's direct sum of the same charges (its own test holds it to the
oracle).  Sources on the diagonal x = y = z, one array for all three coordinates; some
110 GB in all."""
import ctypes

import pytest

from paper_2003_01836_amd import _capi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_sixteen_vectors_of_2_28_sources():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    lib = _capi.load()
    dev = torch.device("cuda:0")
    if torch.cuda.mem_get_info()[0] < 160 * 2 ** 30:
        pytest.skip("needs 160 GiB of free device memory")
    ns, nt, m = 2 ** 28 + 1001, 1000, 16
    g = torch.Generator(device=dev).manual_seed(1080)
    x = torch.rand(ns, dtype=torch.float64, device=dev, generator=g)
    q = torch.empty((m, ns), dtype=torch.float64, device=dev)
    for row in q:
        row.uniform_(-0.5, 0.5, generator=g)
    t = torch.rand((3, nt), dtype=torch.float64, device=dev, generator=g).sub_(2.0)
    got = torch.zeros((m, nt), dtype=torch.float64, device=dev)
    ref = torch.zeros_like(got)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    tp = [ctypes.c_void_p(t[i].data_ptr()) for i in range(3)]
    sp = [ctypes.c_void_p(x.data_ptr())] * 3
    p = bltc.params(theta=0.0, degree=1, leaf_size=65536, batch_size=1000)
    plan = ctypes.c_void_p()
    _capi.check(lib.bltc_plan_create(ctypes.byref(plan), ctypes.byref(p), nt, *tp, ns, *sp, m, stream))
    _capi.check(lib.bltc_plan_execute(plan, ctypes.c_void_p(q.data_ptr()), m, ns,
                                      ctypes.c_void_p(got.data_ptr()), nt, stream))
    torch.cuda.synchronize()
    lib.bltc_plan_destroy(plan)
    bltc.release_memory()
    _capi.check(lib.bltc_direct(ctypes.byref(p), nt, *tp, ns, *sp, ctypes.c_void_p(q.data_ptr()), m, ns,
                                ctypes.c_void_p(ref.data_ptr()), nt, stream))
    # 2.7 10^8 terms of either sign, each below 0.3: partial sums are of the size of the
    # result and every addition rounds them by 2^-53, in the worst case all one way
    # 3e-8 of it, by chance 2e-12
    scale = float(ref.abs().max())
    assert scale > 1.0
    assert float((got - ref).abs().max()) <= 1e-9 * scale
    del x, q
    torch.cuda.empty_cache()
