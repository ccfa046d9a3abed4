"""Sizes of the device blocks that plans take (device_pool), on the host."""
import ctypes

from paper_2003_01836_amd import _capi


def test_block_sizes():
    f = _capi.load().bltc_internal_block_bytes
    f.argtypes, f.restype = [ctypes.c_int64], ctypes.c_int64
    limit = 1 << 31
    for n in [1, 511, 512, 513, 4097, 10 ** 6, 10 ** 8 + 7, limit - 1, limit]:
        assert n <= f(n) <= n + max(511, n // 16)   # steps of 512 bytes at least
    # blocks that the pool never keeps take what was asked for
    for n in [limit + 1, 3 * 10 ** 9 + 1, 16 << 30, (100 << 30) + 8]:
        assert f(n) == n
