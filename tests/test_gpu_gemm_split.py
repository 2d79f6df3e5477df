"""The large fp32 products (three bf16 parts per entry, csrc/ff_gemm_split.hip)
through ff_kron_apply, which takes them where they are the faster route
(tests/test_gemm_route_cpu.py), and by themselves: at tile edges and
remainders, every operand layout, triangular operands, segments, partial sums,
small, large and infinite entries, against fp64."""
import ctypes
import math

import numpy as np
import pytest
import torch

import paper_2609_14706_amd as ffe

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


def _spd(d, seed):
    g = torch.Generator().manual_seed(seed)
    Q = torch.randn(d, d, generator=g, dtype=torch.float64)
    return (Q @ Q.T / d + torch.eye(d, dtype=torch.float64)).float()


def _handle(m, n, batch):
    A, B = _spd(n, 1), _spd(m, 2)
    # as many samples as matrices to apply: the workspace then takes the whole batch in one launch
    G = torch.zeros(batch, m, n, device="cuda")
    return ffe.FlipFlop(G, A0=A.cuda(), B0=B.cuda()), A.double(), B.double()


# rows, columns and k: below, at and above the 128 tile and the 32-wide k
# slice, odd (scalar loads) and multiples of four (16-byte loads)
SHAPES = [(255, 127, 260), (256, 128, 256), (36, 33, 300), (1, 130, 256), (257, 31, 130), (300, 1, 260),
          (264, 200, 70), (520, 132, 80), (520, 516, 40), (2049, 1537, 1)]


@pytest.mark.parametrize("m,n,batch", SHAPES)
def test_products_against_fp64(m, n, batch):
    f, A, B = _handle(m, n, batch)
    X = torch.randn(batch, m, n, generator=torch.Generator().manual_seed(3))
    Y = f.kron_apply(X.cuda()).cpu().double()
    Xd = X.double()
    ref = B @ Xd @ A
    # a product's dropped parts are below 2^-22 of it; a sum over k rounds
    # 6 k / 32 times (random signs: the square root of that counts), plus the
    # rounding of the intermediate and the result
    scale = B.abs() @ Xd.abs() @ A.abs()
    bound = U32 * (4 + 3 + math.sqrt(6 * max(m, n) / 32))
    assert ((Y - ref).abs() / scale).max() <= bound
    # together: two products, each within a few roundings of its sums
    assert float((Y - ref).norm() / ref.norm()) <= 8 * U32
    f.close()


@pytest.mark.parametrize("m,n", [(1024, 1024), (520, 516)])
def test_one_matrix_alone_and_in_a_batch(m, n):
    """The batch may change the route and with it the last bits of a matrix's
    result, no more: both are as near to the exact product as fp32 sums are."""
    f, A, B = _handle(m, n, 40)
    X = torch.randn(40, m, n, generator=torch.Generator().manual_seed(3))
    together, alone = f.kron_apply(X.cuda())[7], f.kron_apply(X[7:8].cuda())[0]
    ref = B @ X[7].double() @ A
    for Y in (together, alone):
        # two products of K / 2 roundings of either sign
        assert float((Y.cpu().double() - ref).norm() / ref.norm()) <= U32 * math.sqrt((m + n) / 2)
    # the same call gives the same bits
    assert torch.equal(alone, f.kron_apply(X[7:8].cuda())[0])
    f.close()


@pytest.mark.parametrize("m,n,batch", [(127, 129, 260), (256, 260, 70), (36, 33, 300), (520, 516, 40)])
def test_triangular_products_against_fp64(m, n, batch):
    f, A, B = _handle(m, n, batch)
    X = torch.randn(batch, m, n, generator=torch.Generator().manual_seed(4))
    Y = f.kron_apply(X.cuda(), inverse=True).cpu().double()
    ref = torch.linalg.solve(B, X.double()) @ torch.linalg.inv(A)
    # condition numbers around 5: the fp32 factorisation's rounding is amplified by them
    assert float((Y - ref).norm() / ref.norm()) <= 1e-5
    f.close()


def _dense(d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    Q = torch.randn(d, d, generator=g, device="cuda", dtype=torch.float64)
    return (Q @ Q.T / d + torch.eye(d, device="cuda", dtype=torch.float64)).float()


# 2048 x 2048: a single matrix takes the split kernel
WIDE_M, WIDE_N = 2048, 2048


def _wide_handle(A, B):
    return ffe.FlipFlop(torch.zeros(1, B.shape[0], A.shape[0], device="cuda"), A0=A, B0=B)


@pytest.mark.parametrize("value", [float(np.finfo(np.float32).max), 3.395e38, -3.3895e38])
def test_entries_near_the_largest_float(value):
    """Finite as long as the sums are: what an fp32 product gives."""
    A, B = _dense(WIDE_N, 1) * 0.1, _dense(WIDE_M, 2) * 0.1
    f = _wide_handle(A, B)
    X = torch.zeros(1, WIDE_M, WIDE_N, device="cuda")
    X[0, 11, 12] = value
    Y = f.kron_apply(X).double()
    ref = B.double() @ X.double() @ A.double()
    # one product per sum and two roundings; the second product (of ordinary
    # numbers) drops parts of up to 2^-24
    assert bool(torch.isfinite(Y).all())
    assert float(((Y - ref).abs() / ref.abs()).max()) <= 6 * U32
    f.close()


def test_infinities_and_nans():
    A, B = _dense(WIDE_N, 1), _dense(WIDE_M, 2)
    f = _wide_handle(A, B)
    X = torch.randn(4, WIDE_M, WIDE_N, generator=torch.Generator().manual_seed(5)).cuda()
    want = f.kron_apply(X[3:].contiguous())
    X[0, 5, 7] = math.inf
    X[1, 6, 8] = -math.inf
    X[2, 7, 9] = math.nan
    Y = f.kron_apply(X)
    # column 7 of B X is infinite with the signs of B's column 5, so row i of
    # the result is infinite with the sign of B[i, 5] A[7, j]
    assert torch.equal(Y[0], (B[:, 5, None] * A[7]).sign() * math.inf)
    assert torch.equal(Y[1], (B[:, 6, None] * A[8]).sign() * -math.inf)
    assert torch.isnan(Y[2]).all()
    assert torch.equal(Y[3], want[0])
    f.close()


# ------------------------------------------------- the kernel by itself
class GemmF32(ctypes.Structure):   # csrc/ff_kernels.hpp
    _fields_ = [(n, ctypes.c_void_p) for n in "ABC"] + [
        (n, ctypes.c_int64) for n in ("lda", "ldb", "ldc", "sA", "sB", "sC", "M", "N", "K")] + [
        ("transA", ctypes.c_int), ("transB", ctypes.c_int), ("alpha", ctypes.c_float), ("beta", ctypes.c_float),
        ("flags", ctypes.c_int), ("kseg", ctypes.c_int64), ("segA", ctypes.c_int64), ("segB", ctypes.c_int64),
        ("ksplit", ctypes.c_int), ("st", ctypes.c_void_p), ("tile", ctypes.c_int)]


K_HI_ROW, K_LO_ROW, K_HI_COL, K_LO_COL, C_LOWER = 1, 2, 4, 8, 16


def _launch(A, B, C, M, N, K, ta=0, tb=0, *, alpha=1.0, beta=0.0, flags=0, seg=None, ksplit=1, deep=False):
    """C = alpha op(A) op(B) + beta C of contiguous device tensors, by launch_gemm_split itself."""
    fn = ffe.load_library()["_ZN2ff17launch_gemm_splitERKNS_7GemmF32EibbP12ihipStream_t"]
    fn.argtypes = [ctypes.POINTER(GemmF32), ctypes.c_int, ctypes.c_bool, ctypes.c_bool, ctypes.c_void_p]
    fn.restype = ctypes.c_int
    st = torch.zeros(4, dtype=torch.int32, device="cuda")
    g = GemmF32(A=A.data_ptr(), B=B.data_ptr(), C=C.data_ptr(), lda=A.shape[-1], ldb=B.shape[-1], ldc=C.shape[-1],
                M=M, N=N, K=K, transA=ta, transB=tb, alpha=alpha, beta=beta, flags=flags, ksplit=ksplit,
                st=st.data_ptr())
    if seg is not None:
        g.kseg = seg
        g.segA, g.segB = A.shape[-2] * seg, B.shape[-2] * seg
    if ksplit > 1:
        g.sC = C.shape[-2] * C.shape[-1]
    vec = all(v % 4 == 0 for v in (g.lda, g.ldb, g.kseg, g.segA, g.segB))
    torch.cuda.synchronize()
    assert fn(ctypes.byref(g), 1, vec, deep, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


def _randn(*shape, seed=0):
    return torch.randn(*shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


def _exact(A, B, ta, tb):
    a = (A.T if ta else A).double().contiguous()
    b = (B.T if tb else B).double().contiguous()
    return a @ b, a.abs() @ b.abs()


def _worst(terms):
    """Bound of |error| / sum |a b|: the dropped products (2^-24 of each at the
    worst), a rounding of the six sums for every 32 of them and of the result."""
    return U32 * (1 + 6 * math.ceil(terms / 32) + 1)


def _typical(K):
    """2-norm error of sums over K products by the fp32 matrix instructions:
    K / 2 roundings of either sign, half a unit each at the most."""
    return U32 * math.sqrt(K / 2)


@pytest.mark.parametrize("deep", [False, True])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(256, 128, 64), (300, 132, 100), (257, 129, 37), (130, 200, 31), (3, 260, 512)])
def test_every_form(M, N, K, ta, tb, deep):
    A = _randn(*((K, M) if ta else (M, K)), seed=1)
    B = _randn(*((N, K) if tb else (K, N)), seed=2)
    C = torch.full((M, N), math.nan, device="cuda")
    _launch(A, B, C, M, N, K, ta, tb, deep=deep)
    ref, scale = _exact(A, B, ta, tb)
    assert float(((C.double() - ref).abs() / scale).max()) <= _worst(K)
    assert float((C.double() - ref).norm() / ref.norm()) <= 2 * U32 + _typical(K)


# a slice, a chunk of the deep form (32 slices) and one more slice, a remainder
@pytest.mark.parametrize("K", [32, 1024, 1056, 2080 + 7])
def test_long_k_with_beta(K):
    M, N = 260, 136
    A, B, C0 = _randn(M, K, seed=1), _randn(N, K, seed=2), _randn(M, N, seed=3)
    C = C0.clone()
    _launch(A, B, C, M, N, K, 0, 1, alpha=-1.0, beta=1.0, deep=True)
    ref, scale = _exact(A, B, 0, 1)
    ref = C0.double() - ref
    assert float(((C.double() - ref).abs() / (scale + C0.abs())).max()) <= _worst(K) + U32
    assert float((C.double() - ref).norm() / ref.norm()) <= 2 * U32 + _typical(K)


@pytest.mark.parametrize("flag,side", [(K_HI_ROW, "A"), (K_LO_ROW, "A"), (K_HI_COL, "B"), (K_LO_COL, "B")])
@pytest.mark.parametrize("d,other", [(600, 150), (257, 300)])
def test_triangular_ranges(flag, side, d, other):
    lower = flag in (K_HI_ROW, K_LO_COL)
    T = _randn(d, d, seed=1)
    T = T.tril() if lower else T.triu()
    X = _randn(d, other, seed=2) if side == "A" else _randn(other, d, seed=2)
    A, B = (T, X) if side == "A" else (X, T)
    M, N = A.shape[0], B.shape[1]
    C = torch.empty(M, N, device="cuda")
    _launch(A.contiguous(), B.contiguous(), C, M, N, d, flags=flag)
    ref, scale = _exact(A, B, 0, 0)
    assert float(((C.double() - ref).abs() / scale.clamp_min(1e-30)).max()) <= _worst(d)


# the symmetric product over stacked samples: tiles on and below the diagonal,
# k in segments (slices within one and across two), split into partial sums
@pytest.mark.parametrize("deep", [False, True])
@pytest.mark.parametrize("d,seg,count,ksplit", [(256, 64, 40, 7), (300, 96, 21, 3), (129, 40, 30, 4), (520, 36, 20, 1),
                                                (64, 128, 9, 2)])
def test_symmetric_product_of_segments(d, seg, count, ksplit, deep):
    X = _randn(count, d, seg, seed=4)
    C = torch.full((ksplit, d, d), math.nan, device="cuda")
    _launch(X, X, C, d, d, count * seg, 0, 1, flags=C_LOWER, seg=seg, ksplit=ksplit, deep=deep)
    x = X.double().permute(1, 0, 2).reshape(d, count * seg)
    ref, scale = x @ x.T.contiguous(), x.abs() @ x.abs().T.contiguous()
    low = torch.ones(d, d, dtype=torch.bool, device="cuda").tril()
    got = C.double().sum(0)
    assert bool(torch.isnan(C[:, ~low]).all())   # nothing above the diagonal is written
    assert float(((got - ref).abs() / scale)[low].max()) <= _worst(count * seg)
    assert float((got - ref)[low].norm() / ref[low].norm()) <= 2 * U32 + _typical(count * seg)


@pytest.mark.parametrize("deep", [False, True])
@pytest.mark.parametrize("power", [-96, -100, -104, -110, -116, -122, -125])
def test_small_entries_keep_their_bits(power, deep):
    """As near to the exact product as fp32 products, down to the smallest
    normal numbers; ordinary rows beside small ones too."""
    M, N, K = 256, 128, 512
    A, B = _randn(M, K, seed=1), _randn(K, N, seed=2)
    A[:100] = torch.ldexp(A[:100], torch.tensor(power))
    C = torch.empty(M, N, device="cuda")
    _launch(A, B, C, M, N, K, deep=deep)
    ref, _ = _exact(A, B, 0, 0)
    for rows in (slice(0, 100), slice(100, None)):
        # the smallest results are subnormal: half of 2^-149 each
        floor = 2.0 ** -150 * math.sqrt(K / 2 * ref[rows].numel())
        assert float((C.double() - ref)[rows].norm()) <= (2 * U32 + _typical(K)) * float(ref[rows].norm()) + floor


@pytest.mark.parametrize("deep", [False, True])
def test_small_second_operand_and_small_products(deep):
    M, N, K = 256, 128, 512
    for pa, pb in ((0, -110), (-60, -60), (60, -115)):
        A = torch.ldexp(_randn(M, K, seed=1), torch.tensor(pa))
        B = torch.ldexp(_randn(K, N, seed=2), torch.tensor(pb))
        C = torch.empty(M, N, device="cuda")
        _launch(A, B, C, M, N, K, deep=deep)
        ref, _ = _exact(A, B, 0, 0)
        floor = 2.0 ** -150 * math.sqrt(6 * K / 32 * ref.numel())
        assert float((C.double() - ref).norm()) <= (2 * U32 + _typical(K)) * float(ref.norm()) + floor


@pytest.mark.parametrize("deep", [False, True])
def test_sums_of_one_term(deep):
    """A diagonal factor: a little more than the one rounding of the fp32 instructions."""
    d, N = 512, 200
    A, B = torch.diag(torch.rand(d, generator=torch.Generator().manual_seed(1)) + 0.5).cuda(), _randn(d, N, seed=2)
    C = torch.empty(d, N, device="cuda")
    _launch(A, B, C, d, N, d, deep=deep)
    ref, _ = _exact(A, B, 0, 0)
    # dropped products at most 2^-24; the sum's rounding 2^-24 where a vector
    # instruction adds the leading product to the lower ones, up to a whole
    # unit (2^-23) where the matrix instruction does (deep); 2^-31 each in the
    # lower parts.  Together: half or whole units, uniform, of a mean number of its binade
    err = (C.double() - ref).abs()
    assert float((err / ref.abs()).max()) <= (3.1 if deep else 2.1) * U32
    assert float(err.norm() / ref.norm()) <= (1.0 if deep else 0.5) * U32
