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


def test_every_slice_of_the_seed_holds_its_statistics(L):
    """2 R floats at the start of every slice of the columns, inside the slice and inside the row."""
    import random
    place = getattr(L, "_ZN3swa16seed_stats_placeEliiiRiS0_")
    place.restype = None
    rng = random.Random(7)
    for _ in range(20000):
        cap = rng.choice((rng.randrange(1, 600), rng.randrange(1, 16385)))
        bound, R = rng.randrange(1, cap + 1), rng.randrange(0, 129)
        pairs = rng.choice((1, 3, 8, 22, 32, 64, 100, 128, 255, 256, 4000))
        G, cols = ctypes.c_int(-1), ctypes.c_int(-1)
        place(ctypes.c_int64(pairs), bound, cap, R, ctypes.byref(G), ctypes.byref(cols))
        if R == 0 or 2 * R > cap:
            assert G.value == 0
            continue
        assert G.value >= 1 and cols.value % 32 == 0
        for g in range(G.value):
            end = cap if g == G.value - 1 else (g + 1) * cols.value
            assert g * cols.value + 2 * R <= end, (pairs, bound, cap, R, G.value, cols.value)


@pytest.mark.parametrize("pairs,bound,cap,R,apart", [
    (32, 8192, 8256, 64, True), (32, 8192, 8192, 64, True), (40, 4200, 4200, 64, True), (40, 4200, 4200, 33, True),
    (128, 4096, 4096, 64, True), (10, 4200, 4200, 64, False), (10, 2200, 2200, 32, False), (64, 1024, 1024, 64, False),
    (64, 1024, 1024, 16, True)])
def test_chains_of_the_statistics_get_workgroups_where_a_slice_can_bring_them_along(L, pairs, bound, cap, R, apart):
    place, rule = L._ZN3swa16seed_stats_placeEliiiRiS0_, L._ZN3swa17seed_chains_apartEiiii
    place.restype, rule.restype = None, ctypes.c_bool
    G, cols = ctypes.c_int(), ctypes.c_int()
    place(ctypes.c_int64(pairs), bound, cap, R, ctypes.byref(G), ctypes.byref(cols))
    assert rule(G, cols, cap, R) is apart
    for g in range(G.value if apart else 0):          # 8 R floats at the start of every slice, inside it and inside the row
        assert g * cols.value + 8 * R <= (cap if g == G.value - 1 else (g + 1) * cols.value)


@pytest.mark.parametrize("pairs,least", [(1, 1024), (32, 1024), (33, 1536), (64, 1536), (65, 2048), (128, 2048)])
def test_split_rows_where_three_launches_pay(L, pairs, least):
    rule = L._ZN3swa12split_factorElibi
    for row in (128, 256, 512):
        for stated in (False, True):
            line = least if stated and row >= 256 else 2048
            assert rule(ctypes.c_int64(pairs), line - 1, ctypes.c_bool(stated), row) == 1, (row, stated)
            assert rule(ctypes.c_int64(pairs), line, ctypes.c_bool(stated), row) > 1, (row, stated)
    assert rule(ctypes.c_int64(129), 16384, ctypes.c_bool(True), 512) == 1
