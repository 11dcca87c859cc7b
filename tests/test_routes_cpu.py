"""The host's choice between forms of a call, where a wrong line costs time and no result shows it: the library's own rules at
the sizes that were measured."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def L():
    import os
    from paper_2403_17312_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    return ctypes.CDLL(binding.LIB_PATH)


@pytest.mark.parametrize("pairs,bound,R,two", [
    (32, 1023, 64, False), (32, 1024, 64, True), (64, 1024, 16, True), (64, 8192, 128, True),
    (96, 1024, 16, False), (96, 4096, 128, False), (128, 2048, 64, False), (128, 4096, 64, True), (128, 8192, 128, False),
    (129, 16384, 16, False), (160, 8192, 64, False), (224, 1024, 64, False), (224, 8192, 128, False), (250, 4096, 64, False)])
def test_seed_takes_two_launches_only_where_they_pay(L, pairs, bound, R, two):
    rule = getattr(L, "_ZN3swa11seed_in_twoElibi")
    rule.restype = ctypes.c_bool
    assert rule(ctypes.c_int64(pairs), bound, ctypes.c_bool(True), R) is two
    assert rule(ctypes.c_int64(pairs), bound, ctypes.c_bool(False), R) is (two and pairs <= 64)
