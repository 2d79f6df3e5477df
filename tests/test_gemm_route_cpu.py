"""The rule that sends an fp32 product to 64 x 64 or 128 x 128 tiles of fp32
instructions or to 256 x 128 tiles of three-part bf16 products
(csrc/ff_gemm_f32.hip), at sizes where the measured times lie well apart."""
import ctypes

import pytest

import paper_2609_14706_amd as ffe
from test_gpu_gemm_split import C_LOWER, K_HI_COL, K_HI_ROW, GemmF32


class Route(ctypes.Structure):
    _fields_ = [("tile", ctypes.c_int), ("us", ctypes.c_double)]


def _route(M, N, K, flags=0, batch=1, ksplit=1, tile=0, vec=True, ld=None):
    fn = ffe.load_library()["_ZN2ff10gemm_routeERKNS_7GemmF32Eib"]
    fn.argtypes, fn.restype = [ctypes.POINTER(GemmF32), ctypes.c_int, ctypes.c_bool], Route
    ld = K if ld is None else ld
    r = fn(GemmF32(M=M, N=N, K=K, flags=flags, ksplit=ksplit, tile=tile, lda=ld, ldb=ld), batch, vec)
    return r.tile, r.us


CASES = [  # tile, measured us, sizes, flags, batch, parts of k
    (64, 22, 16, 16, 16, 0, 2048, 1), (64, 23, 64, 64, 64, 0, 2048, 1), (64, 374, 256, 8192, 8192, 0, 1, 1),
    (64, 190, 512, 4096, 4096, 0, 1, 1), (64, 32, 1024, 1024, 1024, 0, 1, 1), (64, 12, 530, 192, 192, 0, 2, 1),
    (64, 86, 1500, 1500, 1500, K_HI_ROW, 1, 1), (64, 109, 2048, 2048, 2048, K_HI_ROW, 1, 1),
    (64, 47, 262144, 64, 64, K_HI_COL, 1, 1), (64, 25, 16384, 256, 256, K_HI_COL, 1, 1),
    (64, 25, 64, 64, 131072, C_LOWER, 1, 256), (64, 59, 192, 192, 65536, C_LOWER, 1, 170),
    (128, 52, 128, 128, 128, 0, 1024, 1), (128, 85, 128, 256, 256, 0, 512, 1), (128, 68, 100, 100, 100, 0, 1000, 1),
    (256, 236, 2000, 3000, 3000, 0, 1, 1), (256, 132, 1500, 1500, 1500, 0, 2, 1),
    (256, 158, 2048, 2048, 2048, 0, 1, 1), (256, 90, 1024, 1024, 1024, 0, 8, 1),
    (256, 105, 512, 512, 512, 0, 64, 1), (256, 66, 256, 256, 256, 0, 256, 1),
    (256, 205, 2600, 2600, 2600, K_HI_ROW, 1, 1), (256, 50, 512, 512, 512, K_HI_ROW, 32, 1),
    (256, 184, 65536, 512, 512, K_HI_COL, 1, 1), (256, 60, 65536, 256, 256, K_HI_COL, 1, 1),
    (256, 81, 256, 256, 65536, C_LOWER, 1, 170), (256, 666, 1024, 1024, 65536, C_LOWER, 1, 14)]


@pytest.mark.parametrize("case", CASES)
def test_route(case):
    want, us, M, N, K, flags, batch, ksplit = case
    tile, expected = _route(M, N, K, flags, batch, ksplit)
    assert tile == want
    assert us / 1.5 < expected < us * 1.5   # the fit's largest misses here are a third


def test_a_lower_triangle_of_one_tile_is_not_split():
    for d, parts in ((64, 256), (128, 64), (128, 256)):
        assert _route(d, d, 131072, C_LOWER, 1, parts)[0] in (64, 128)


def test_forms():
    big = (8192, 8192, 8192)
    assert _route(*big)[0] == 256 and _route(*big, vec=False)[0] == 256
    assert _route(*big, tile=64)[0] == 64 and _route(*big, tile=128)[0] == 128
    assert _route(*big, ld=1 << 23)[0] == 256 and _route(*big, ld=(1 << 23) + 1)[0] != 256   # 32-bit offsets in a slice
