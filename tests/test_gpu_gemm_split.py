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


def test_extreme_values():
    """Infinities, NaNs, values that round to a bf16 infinity, tiny values:
    as in an fp32 product with dense operands."""
    m, n, batch = 128, 132, 256
    f, A, B = _handle(m, n, batch)
    X = torch.randn(batch, m, n, generator=torch.Generator().manual_seed(5))
    X[3, 5, 7] = math.inf
    X[4, 6, 8] = -math.inf
    X[5, 7, 9] = math.nan
    X[6] *= 1e-36
    X[7] = 0.0
    X[7, 11, 12] = float(np.finfo(np.float32).max)
    Y = f.kron_apply(X.cuda()).cpu()
    ok = torch.ones(batch, dtype=torch.bool)
    ok[3:6] = False
    assert torch.isfinite(Y[ok][[0, 1, 2, 3, 5]]).all()
    assert not torch.isfinite(Y[3:6]).all(dim=2).any()   # every entry's sum meets the non-finite value
    assert torch.isnan(Y[5]).all()
    ref = B @ X[6].double() @ A
    # entries below 2^-126 * 2^16 lose low parts, which sit under fp32's smallest numbers
    assert float((Y[6].double() - ref).norm() / ref.norm()) <= 1e-3
    r7 = B @ X[7].double() @ A
    fin = r7.abs() < 3e38
    t = B[:, 11].abs().max() * float(np.finfo(np.float32).max) < 3.4e38
    if t:
        assert ((Y[7].double() - r7).abs()[fin] <= 1e-6 * r7.abs().max()).all()
    f.close()
