"""The fp32 products on fp32 instructions (csrc/ff_gemm_f32.hip) by
themselves: 64 x 64 and 128 x 128 tiles at their edges, every operand layout,
triangular ranges, segments and partial sums, against fp64 and each other."""
import ctypes

import pytest
import torch

import paper_2609_14706_amd as ffe
from test_gpu_gemm_split import C_LOWER, K_HI_COL, K_HI_ROW, K_LO_COL, K_LO_ROW, GemmF32, U32, _exact, _randn

pytestmark = pytest.mark.gpu


def _launch(tile, A, B, C, M, N, K, ta=0, tb=0, *, alpha=1.0, beta=0.0, flags=0, seg=None, ksplit=1):
    fn = ffe.load_library()["_ZN2ff15launch_gemm_f32ERKNS_7GemmF32EiP12ihipStream_t"]
    fn.argtypes, fn.restype = [ctypes.POINTER(GemmF32), ctypes.c_int, ctypes.c_void_p], ctypes.c_int
    st = torch.zeros(4, dtype=torch.int32, device="cuda")
    g = GemmF32(A=A.data_ptr(), B=B.data_ptr(), C=C.data_ptr(), lda=A.shape[-1], ldb=B.shape[-1], ldc=C.shape[-1],
                M=M, N=N, K=K, transA=ta, transB=tb, alpha=alpha, beta=beta, flags=flags, ksplit=ksplit,
                kseg=K, st=st.data_ptr(), tile=tile)
    if seg is not None:
        g.kseg, g.segA, g.segB = seg, A.shape[-2] * seg, B.shape[-2] * seg
    if ksplit > 1:
        g.sC = C.shape[-2] * C.shape[-1]
    torch.cuda.synchronize()
    assert fn(ctypes.byref(g), 1, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


def _both(shape, *args, start=None, **kw):
    out = []
    for tile in (64, 128):
        C = torch.full(shape, float("nan"), device="cuda") if start is None else start.clone()
        _launch(tile, *args[:2], C, *args[2:], **kw)
        out.append(C)
    return out


def _check(C, ref, scale, K):
    # K / 2 roundings of at most a unit of the sum of magnitudes, and two more
    assert float(((C.double() - ref).abs() / scale.clamp_min(1e-30)).max()) <= U32 * (K / 2 + 2)


@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (129, 132, 100), (64, 65, 31), (1, 260, 33), (200, 127, 96)])
def test_every_form(M, N, K, ta, tb):
    A = _randn(*((K, M) if ta else (M, K)), seed=1)
    B = _randn(*((N, K) if tb else (K, N)), seed=2)
    C0 = _randn(M, N, seed=3)
    ref, scale = _exact(A, B, ta, tb)
    small, large = _both((M, N), A, B, M, N, K, ta, tb)
    _check(small, ref, scale, K)
    assert torch.equal(small, large)   # the same sums in the same order
    small, large = _both((M, N), A, B, M, N, K, ta, tb, alpha=-1.0, beta=1.0, start=C0)
    _check(small, C0.double() - ref, scale + C0.abs(), K)
    assert torch.equal(small, large)


@pytest.mark.parametrize("flag", [K_HI_ROW, K_LO_ROW, K_HI_COL, K_LO_COL])
def test_triangular_ranges(flag):
    d, other = 300, 150
    T = _randn(d, d, seed=1)
    T = (T.tril() if flag in (K_HI_ROW, K_LO_COL) else T.triu()).contiguous()
    left = flag in (K_HI_ROW, K_LO_ROW)
    X = _randn(d, other, seed=2) if left else _randn(other, d, seed=2)
    A, B = (T, X) if left else (X, T)
    shape = (d, other) if left else (other, d)
    ref, scale = _exact(A, B, 0, 0)
    for C in _both(shape, A, B, *shape, d, flags=flag):
        _check(C, ref, scale, d)


@pytest.mark.parametrize("d,seg,count,ksplit", [(128, 64, 40, 7), (130, 96, 21, 3), (100, 40, 30, 4), (64, 128, 9, 2),
                                                (128, 1024, 40, 2)])   # the last: more than 16384 k a workgroup
def test_symmetric_product_of_segments(d, seg, count, ksplit):
    X = _randn(count, d, seg, seed=4)
    x = X.double().permute(1, 0, 2).reshape(d, count * seg)
    ref, scale = x @ x.T.contiguous(), x.abs() @ x.abs().T.contiguous()
    low = torch.ones(d, d, dtype=torch.bool, device="cuda").tril()
    for C in _both((ksplit, d, d), X, X, d, d, count * seg, 0, 1, flags=C_LOWER, seg=seg, ksplit=ksplit):
        assert bool(torch.isnan(C[:, ~low]).all())   # nothing above the diagonal is written
        _check(C.double().sum(0)[low], ref[low], scale[low], count * seg)
