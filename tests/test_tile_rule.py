"""The tiles of an integral, by the rules that the library plans them with."""
import ctypes as C

import pytest

import paper_1408_6373_amd as cc

FP64, FP32 = 0, 1


def _tiles(n, prec, dN, resident=8, bs=256, ncu=256, per_cu=3, refined=True):
    rule = cc._lib["_ZN5ccuba11single_tileExxiiixib"]
    rule.argtypes = [C.c_longlong, C.c_longlong, C.c_int, C.c_int, C.c_int, C.c_longlong, C.c_int,
                     C.c_bool]
    rule.restype = C.c_longlong
    P = rule(n, bs, ncu, per_cu, prec, dN, resident, refined)
    assert P > 0 and P % bs == 0
    return -(-n // P)


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("dN", [2, 1024, 4096])
def test_no_more_tiles_than_blocks(prec, dN):
    for n in (2, 255, 65536, 65537, 10**6, 10**7, 2**32 - 1):
        for per_cu in (1, 2, 3, 16):
            assert _tiles(n, prec, dN, per_cu=per_cu) <= 256 * per_cu
            assert _tiles(n, prec, dN, per_cu=per_cu, resident=1) <= 256
        # a pass alone: a tile per block of points; up to 64 for a refine launch
        assert n > 65536 or _tiles(n, prec, dN, refined=False) == -(-n // 256)
        assert n > 65536 or _tiles(n, prec, dN) <= 64


@pytest.mark.parametrize("n,prec,dN,resident,per_cu", [
    (10**6, FP64, 1024, 3, 1), (2 * 10**6, FP64, 1024, 3, 1), (4 * 10**6, FP64, 1024, 3, 2),
    (10**6, FP32, 1024, 3, 2), (4 * 10**6, FP32, 1024, 3, 2), (10**7, FP32, 1024, 3, 3),
    (3 * 10**6, FP64, 1536, 3, 1), (10**7, FP64, 4096, 1, 1), (10**6, FP32, 4096, 1, 1)])
def test_tiles_follow_the_measured_best(n, prec, dN, resident, per_cu):
    # the fastest of 1, 2 and 3 tiles per compute unit, or within 2% of it, as measured
    assert 256 * (per_cu - 1) < _tiles(n, prec, dN, resident) <= 256 * per_cu


@pytest.mark.parametrize("setting,sizes", [(2048, {2048, 4096, 16384, 65536}),
                                           (4096, {4096, 16384, 65536}),
                                           (65536, {4096, 16384, 65536}),
                                           (100, {100, 4096, 16384, 65536})])
def test_autotuner_tries_the_setting_it_replaces(setting, sizes):
    f = cc._lib["_ZN5ccuba16batch_tile_sizesExPx"]
    f.argtypes = [C.c_longlong, C.POINTER(C.c_longlong)]
    f.restype = C.c_int
    out = (C.c_longlong * 4)()
    n = f(setting, out)
    assert n == len(sizes) and set(out[:n]) == sizes


@pytest.mark.parametrize("total,dN,lo,hi", [
    (8 * 10**6, 2432, 12288, 16384),    # long rows: two tiles per compute unit
    (6.8 * 10**6, 1408, 12288, 16384),
    (4.3 * 10**6, 2100, 6144, 10240),
    (5 * 10**6, 175, 5120, 8192),       # short rows: three
    (10**6, 1024, 2048, 2048),          # the setting's smallest
    (2.7 * 10**7, 2700, 16384, 16384),  # no more than a full tile
    (3 * 10**8, 1024, 40000, 65536)])   # or eight tiles a block
def test_batch_tiles_follow_the_measured_best(total, dN, lo, hi):
    f = cc._lib["_ZN5ccuba10batch_tileExdxxii"]
    f.argtypes = [C.c_longlong, C.c_double, C.c_longlong, C.c_longlong, C.c_int, C.c_int]
    f.restype = C.c_longlong
    P = f(int(total), float(total) * dN, 2048, 256, 256, 3)
    assert P % 256 == 0 and lo <= P <= hi
    assert f(int(total), float(total) * dN, 131072, 256, 256, 3) == 131072  # a larger setting
