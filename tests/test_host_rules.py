"""Rules that the host decides launches by, on the CPU (built into tests/native/libhfe_exact_check.so)."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libhfe_exact_check.so")
if not os.path.exists(LIB):  # pragma: no cover
    pytest.fail(f"{LIB} is missing: build it with `python paper_2601_17561_amd/build.py`", pytrace=False)
_L = ctypes.CDLL(LIB)
_i64 = ctypes.c_int64
_L.xc_gemm_splits.argtypes = [_i64, _i64, _i64, _i64, ctypes.c_int, _i64]
_L.xc_gemm_splits.restype = ctypes.c_int

_ints = ctypes.POINTER(ctypes.c_int32)
_L.xc_per_device.argtypes = [_ints, ctypes.c_int32, _ints, _ints, _ints]
_L.xc_per_device.restype = None
_L.xc_tuned_tile.argtypes = [ctypes.POINTER(_i64), ctypes.c_int32, ctypes.c_int, _i64, ctypes.c_int]
_L.xc_tuned_tile.restype = ctypes.c_int
_L.xc_tune_bucket.argtypes = [_i64]
_L.xc_tune_bucket.restype = _i64

DIGIT, N2, RNS = 0, 1, 2
TILE = 64 << 10  # bytes of one tile's results, every form


# workgroups, K-blocks, columns -> parts by the measured times: the chip nearly empty, half full, a few over a round
@pytest.mark.parametrize("form,tiles,KB,cols,parts", [
    (DIGIT, 6, 128, 48, 8), (DIGIT, 52, 128, 48, 4), (DIGIT, 520, 328, 64, 2), (DIGIT, 1040, 328, 128, 2),
    (DIGIT, 1288, 328, 128, 2), (DIGIT, 1592, 328, 128, 1), (N2, 84, 128, 128, 3), (N2, 156, 128, 128, 1),
    (N2, 156, 128, 16, 3), (N2, 630, 328, 75, 2), (N2, 1224, 328, 128, 1), (RNS, 154, 128, 200, 1),
    (RNS, 286, 128, 16, 2), (RNS, 286, 128, 256, 1), (RNS, 2145, 328, 64, 1), (RNS, 2145, 328, 256, 1)])
def test_parts_of_measured_contractions(form, tiles, KB, cols, parts):
    assert _L.xc_gemm_splits(tiles, 256, KB, cols, form, tiles * TILE) == parts


@pytest.mark.parametrize("form", [DIGIT, N2, RNS])
@pytest.mark.parametrize("cus", [256, 304])
def test_parts_are_few_and_their_buffer_bounded(form, cus):
    for KB in (1, 15, 32, 145, 328, 1024, 2048):
        for tiles, cols in ((t, c) for t in range(1, 20 * cus, 7) for c in (16, 100)):
            s = _L.xc_gemm_splits(tiles, cus, KB, cols, form, tiles * TILE)
            assert 1 <= s <= max(1, KB // 16) and s <= (16 if tiles <= cus else 4)
            assert s == 1 or s * tiles * TILE <= 256 << 20


def test_each_device_has_its_own_value_asked_for_once():
    def call(devs, counts):
        n, arr = len(devs), lambda v: (ctypes.c_int32 * len(v))(*v)
        out, asked = arr([0] * n), arr([0] * n)
        _L.xc_per_device(arr(devs), n, arr(counts), out, asked)
        return list(out), list(asked)

    assert call([0, 1, 0, 1, 0], [256, 304]) == ([256, 304, 256, 304, 256], [1, 2, 2, 2, 2])
    assert call([1, 1, -1, -1], [256, 0]) == ([0, 0, 0, 0], [1, 2, 3, 4])  # a failed query is not kept
    assert call([70, 70], [0] * 70 + [128]) == ([128, 128], [1, 2])        # beyond the table: asked each time


# entries (level, bucket, tile): the nearest of the level, and calls of up to 32 columns apart from larger ones
@pytest.mark.parametrize("table,level,d3,tile", [
    ([], 3, 16, 99), ([(3, 512, 5)], 3, 16, 99), ([(3, 512, 5)], 3, 33, 5), ([(3, 32, 12)], 3, 16, 12),
    ([(3, 32, 12)], 3, 33, 99), ([(3, 32, 12), (3, 64, 4), (3, 1024, 5)], 3, 128, 4), ([(2, 64, 4)], 3, 64, 99),
    ([(3, 0, 4), (3, -8, 4)], 3, 16, 99)])
def test_tuned_tiles_serve_calls_of_their_kind(table, level, d3, tile):
    flat = [x for e in table for x in e]
    assert _L.xc_tuned_tile((_i64 * len(flat))(*flat), len(table), level, d3, 99) == tile


def test_tuning_buckets_separate_the_narrow_tile():
    assert [_L.xc_tune_bucket(d) for d in (1, 32, 33, 64, 65, 512, 513)] == [32, 32, 64, 64, 128, 512, 1024]
