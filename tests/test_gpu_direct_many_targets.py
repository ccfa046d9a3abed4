"""The direct sum of more targets than one launch takes (2^30 is where a grid of 256
threads per 64 targets reaches the 2^32 threads a dimension may have): targets on the
diagonal x = y = z, so one array of 8 GiB serves as all three coordinates, against the
kernel values formed by torch in FP64, over the whole array in parts."""
import ctypes
import math

import pytest

from paper_2003_01836_amd import _capi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
def test_direct_beyond_2_30_targets(noalloc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_01836_amd as bltc
    lib = _capi.load()
    dev = torch.device("cuda:0")
    nt = 2 ** 30 + 65
    if torch.cuda.mem_get_info()[0] < 40 * 2 ** 30:
        pytest.skip("needs 20 GiB of device memory")
    x = torch.arange(nt, dtype=torch.float64, device=dev)
    x.add_(1.0)
    phi = torch.empty(nt, dtype=torch.float64, device=dev)
    s = torch.tensor([[0.0], [-2.0]], dtype=torch.float64, device=dev).repeat(1, 3).t().contiguous()
    q = torch.tensor([2.0, -0.5], dtype=torch.float64, device=dev)
    ptr = [ctypes.c_void_p(r.data_ptr()) for r in (x, x, x, s[0], s[1], s[2], q, phi)]
    p = bltc.params()
    fn = lib.bltc_direct_noalloc if noalloc else lib.bltc_direct
    _capi.check(fn(ctypes.byref(p), nt, *ptr[:3], 2, *ptr[3:6], ptr[6], 1, 2, ptr[7], nt,
                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    for i in range(0, nt, 2 ** 27):
        d = x[i:i + 2 ** 27]
        ref = (2.0 / d - 0.5 / (d + 2.0)) / math.sqrt(3.0)
        # FP64 bar of the suite, relative to each value (two terms of one sign's size)
        assert torch.all((phi[i:i + 2 ** 27] - ref).abs() <= 1e-12 * ref)
    del x, phi, ref, d
    torch.cuda.empty_cache()
