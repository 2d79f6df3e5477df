"""The rule that sends an fp32 product to 64 x 64 tiles of fp32 instructions or
to 256 x 128 tiles of three-part bf16 products (csrc/ff_gemm_f32.hip), at sizes
where the measured times of the two routes lie well apart."""
import ctypes

import pytest

import paper_2609_14706_amd as ffe
from test_gpu_gemm_split import C_LOWER, K_HI_COL, K_HI_ROW, GemmF32


def _takes_split(M, N, K, flags=0, batch=1, ksplit=1, tile=0, vec=True, ld=None):
    fn = ffe.load_library()["_ZN2ff16gemm_takes_splitERKNS_7GemmF32Eib"]
    fn.argtypes, fn.restype = [ctypes.POINTER(GemmF32), ctypes.c_int, ctypes.c_bool], ctypes.c_bool
    ld = K if ld is None else ld
    return fn(GemmF32(M=M, N=N, K=K, flags=flags, ksplit=ksplit, tile=tile, lda=ld, ldb=ld), batch, vec)


SMALL = [  # sizes, flags, batch, ksplit
    (16, 16, 16, 0, 2048, 1), (64, 64, 64, 0, 2048, 1), (128, 128, 128, 0, 1024, 1), (128, 16384, 16384, 0, 1, 1),
    (256, 8192, 8192, 0, 1, 1), (512, 4096, 4096, 0, 1, 1), (1024, 1024, 1024, 0, 1, 1), (530, 192, 192, 0, 2, 1),
    (1500, 1500, 1500, K_HI_ROW, 1, 1), (2048, 2048, 2048, K_HI_ROW, 1, 1), (262144, 64, 64, K_HI_COL, 1, 1),
    (16384, 256, 256, K_HI_COL, 1, 1), (64, 64, 131072, C_LOWER, 1, 256), (128, 128, 131072, C_LOWER, 1, 256),
    (192, 192, 65536, C_LOWER, 1, 170)]
LARGE = [
    (2000, 3000, 3000, 0, 1, 1), (1500, 1500, 1500, 0, 2, 1), (2048, 2048, 2048, 0, 1, 1), (1024, 1024, 1024, 0, 8, 1),
    (512, 512, 512, 0, 64, 1), (256, 256, 256, 0, 256, 1), (2600, 2600, 2600, K_HI_ROW, 1, 1),
    (512, 512, 512, K_HI_ROW, 32, 1), (65536, 512, 512, K_HI_COL, 1, 1), (65536, 256, 256, K_HI_COL, 1, 1),
    (256, 256, 65536, C_LOWER, 1, 170), (1024, 1024, 65536, C_LOWER, 1, 14), (22528, 22528, 2048, C_LOWER, 1, 1)]


@pytest.mark.parametrize("want,case", [(False, c) for c in SMALL] + [(True, c) for c in LARGE])
def test_route(want, case):
    M, N, K, flags, batch, ksplit = case
    assert _takes_split(M, N, K, flags, batch, ksplit) is want


def test_refused_forms():
    big = (8192, 8192, 8192)
    assert _takes_split(*big) and _takes_split(*big, vec=False)
    assert not _takes_split(*big, tile=64)
    assert _takes_split(*big, ld=1 << 23) and not _takes_split(*big, ld=(1 << 23) + 1)   # 32-bit offsets in a slice
    assert not _takes_split(8192, 8256, 8192, flags=C_LOWER)                             # the triangle of a square
