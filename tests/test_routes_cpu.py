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
    assert L._ZN3swa17split_piece_bytesEl(ctypes.c_int64(pairs)) == (64 if pairs <= 64 else 128)


UNORDERED, ORDERED, SHARED, TWO_CALL = 1 | 2, 1, 1 | 2 | 4, 0


def threads(L, pairs, bound, flags, dtype, d, stated=True, ring=False, cap=16384, w=64):
    from paper_2403_17312_amd import binding as B
    assert UNORDERED == B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED and SHARED == UNORDERED | B.SWA_HEAD_SHARED
    rule = L._ZN3swa20decode_block_threadsERK10swa_paramslib
    p = B.make_params(pairs, 1, d, cap, w, 8000, dtype, len_bound=bound if stated else 0, flags=flags)
    return rule(ctypes.byref(p), ctypes.c_int64(pairs), bound, ctypes.c_bool(ring))


@pytest.mark.parametrize("flags,dtype,d,pairs,least", [
    (UNORDERED, "f16", 128, 4, 4481), (UNORDERED, "bf16", 64, 4096, 4481), (UNORDERED, "f32", 64, 300, 4481), (UNORDERED, "f32", 128, 4096, 3585),
    (SHARED, "f16", 128, 4096, 3585), (SHARED, "f32", 128, 12, 3585), (SHARED, "f32", 64, 12, 3585), (SHARED, "bf16", 64, 256, 3585), (SHARED, "bf16", 64, 512, 3841),
    (ORDERED, "f16", 128, 256, 2049), (ORDERED, "bf16", 64, 4, 2049), (ORDERED, "f32", 128, 257, 4481), (ORDERED, "bf16", 64, 4096, 4481),
    (TWO_CALL, "f16", 128, 128, 8961), (TWO_CALL, "f32", 128, 8, 8961), (TWO_CALL, "bf16", 64, 129, 0), (TWO_CALL, "f32", 64, 512, 0)])
def test_1024_threads_from_one_line_on(L, flags, dtype, d, pairs, least):
    """Up to the longest cache that a form takes, under a stated bound, whatever the window; no line without a bound or for the strict window."""
    import torch
    dt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    top = {UNORDERED: 7168, SHARED: 7168, ORDERED: 9216, TWO_CALL: 16384}[flags]
    for bound in sorted({257, 600, 1023, 1024, 1025, 2000, 2048, 2049, 3000, 3585, 4480, 4481, top, max(1, least - 1), least or top}):
        if bound > top:
            continue
        for w in (4, 64):
            assert (threads(L, pairs, bound, flags, dt, d, w=w) == 1024) == (0 < least <= bound), (bound, w)
        assert threads(L, pairs, bound, flags, dt, d, stated=False, cap=bound) <= 512
        if flags == UNORDERED:
            assert threads(L, pairs, bound, flags, dt, d, ring=True) <= 512


@pytest.mark.parametrize("flags,ring,dtype,d,pairs,least", [
    (UNORDERED, False, "f16", 128, 96, 257), (UNORDERED, False, "f16", 128, 97, 385), (UNORDERED, False, "f32", 64, 128, 385),
    (UNORDERED, False, "f32", 128, 128, 257), (UNORDERED, False, "bf16", 64, 4, 385), (SHARED, False, "bf16", 64, 84, 385), (SHARED, False, "f16", 128, 8, 257),
    (TWO_CALL, False, "bf16", 64, 128, 385), (TWO_CALL, False, "f16", 128, 128, 385), (ORDERED, False, "bf16", 64, 128, 257),
    (ORDERED, False, "f16", 128, 128, 257), (UNORDERED, True, "bf16", 64, 128, 257), (UNORDERED, True, "f32", 64, 97, 257),
    (UNORDERED, False, "f32", 128, 129, 1024), (ORDERED, False, "f16", 128, 129, 1024), (UNORDERED, True, "f16", 128, 129, 1024)])
def test_512_threads_where_few_pairs_gain(L, flags, ring, dtype, d, pairs, least):
    import torch
    dt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    for bound in (64, 256, 257, 300, 384, 385, 1023, 1024, 1500):
        assert threads(L, pairs, bound, flags, dt, d, ring=ring) == (512 if bound >= least else 256), bound
        assert threads(L, pairs, bound, flags, dt, d, stated=False, ring=ring, cap=bound) == (512 if bound >= 1024 else 256), bound


def test_threads_of_the_8_bit_cache_go_with_pairs_and_bound(L):
    import torch
    for stated in (False, True):
        for pairs in (4, 128, 1023, 1024, 4096):
            for bound in (64, 300, 1023, 1024, 7168):
                got = threads(L, pairs, bound, UNORDERED | 8, torch.float16, 128, stated=stated, cap=bound)
                assert got == (128 if pairs >= 1024 and bound < 1024 else 256), (stated, pairs, bound)
