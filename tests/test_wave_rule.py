"""Waves of an interaction workgroup (group_log_waves), on the host: full and short
groups on both sides of every line of the rule, the bounds of a kernel and the lanes a
caller asks for."""
import ctypes

import pytest

from paper_2003_01836_amd import _capi


def waves(targets, groups, asked=1, most=16, early=False):
    f = _capi.load().bltc_internal_waves
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32]
    f.restype = ctypes.c_int32
    return f(targets, groups, asked, most, int(early))


@pytest.mark.parametrize("targets,groups,early,want", [
    (1, 1, False, 16), (1500, 64, True, 16), (30011, 512, True, 16),
    (64 * 511, 511, False, 16), (64 * 511 + 1, 512, False, 8),
    (30000, 1300, False, 16), (30000, 1536, False, 8),            # 23 and 20 targets a group
    (100003, 2048, False, 8), (500000, 8192, False, 8), (500000, 7168, True, 4),
    (500000, 7167 + 650, True, 4), (458000, 7167, True, 8),
    (64 * 8192, 8192, False, 4), (1000000, 15872, True, 4), (1100000, 20480, False, 4),
    (64 * 32767, 32767, True, 4), (64 * 32768, 32768, False, 1), (64 * 10 ** 6, 10 ** 6, True, 1),
    # groups less than half full
    (30000, 2047, False, 8), (30000, 2048, False, 4), (30000, 4096, True, 4),
    (100000, 7167, False, 4), (100000, 7168, False, 1), (100000, 31000, True, 1),
    (1000000, 32768, False, 1), (1000000, 31250, False, 4)])
def test_waves_of_a_workgroup(targets, groups, early, want):
    assert waves(targets, groups, early=early) == want


def test_bounds_and_lanes_asked_for():
    assert waves(1, 1, most=8) == 8
    assert waves(1, 1, most=1) == 1
    assert [waves(10 ** 8, 10 ** 7, asked=a) for a in (1, 2, 4)] == [1, 2, 4]
    assert [waves(10 ** 6, 16000, asked=a) for a in (1, 2, 4)] == [4, 4, 4]
    assert waves(10 ** 8, 10 ** 7, asked=4, most=2) == 2


def test_within_the_threads_of_a_grid():
    # 2^32 threads a dimension at most, a wave has 64
    assert waves(2 ** 27, 2 ** 23, asked=4) == 4
    assert waves(2 ** 27, 2 ** 24, asked=4) == 2
    assert waves(2 ** 28, 2 ** 25, asked=4) == 1
