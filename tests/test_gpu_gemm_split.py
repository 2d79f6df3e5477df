"""The large fp32 products (three bf16 parts per entry, csrc/ff_gemm_split.hip)
through ff_kron_apply, which takes them once a launch has 192 tiles of
128 x 128 (400 with a triangular operand of more than one tile): at tile edges
and remainders, both operand layouts, triangular operands, against fp64."""
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
          (264, 200, 70), (520, 132, 80)]


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


@pytest.mark.parametrize("m,n,batch", [(127, 129, 260), (256, 260, 70), (36, 33, 300)])
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


# 1536 x 2048: 192 tiles of one matrix
WIDE_M, WIDE_N = 1536, 2048


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
    # numbers) drops parts of up to 2^-22
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
