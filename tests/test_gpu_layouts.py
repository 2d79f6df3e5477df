"""Layouts that take another route inside the library: factorisations whose
width is no multiple of four (padded rows), samples of odd width, tokens that
are read where the caller has them, the tokens' identity start, and the
allocation-free entry point at its scratch limit; against fp64 or the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_14706_amd as ffe

pytestmark = pytest.mark.gpu


def _spd(d, seed):
    g = torch.Generator().manual_seed(seed)
    Q = torch.randn(d, d, generator=g, dtype=torch.float64)
    return (Q @ Q.T / d + torch.eye(d, dtype=torch.float64)).float()


def _samples(N, m, n, dtype=torch.float32, seed=7):
    g = torch.Generator().manual_seed(seed)
    s = torch.arange(1, n + 1) ** -0.4
    return (torch.randn(N, m, n, generator=g) * s).to(dtype)


# one leaf, a leaf and a remainder of 1, 2 and 3 columns, several panels
@pytest.mark.parametrize("m,n", [(127, 129), (130, 131), (257, 386), (515, 129), (3, 641)])
def test_factorisation_of_odd_width(gpu, m, n):
    A, B = _spd(n, 1), _spd(m, 2)
    f = ffe.FlipFlop(torch.zeros(1, m, n, device=gpu), A0=A.to(gpu), B0=B.to(gpu))
    X = torch.randn(2, m, n, generator=torch.Generator().manual_seed(3))
    Y = f.kron_apply(X.to(gpu), inverse=True).cpu().double()
    ref = torch.linalg.solve(B.double(), X.double()) @ torch.linalg.inv(A.double())
    # condition numbers around 5; fp32 factorisation and products
    assert float((Y - ref).norm() / ref.norm()) <= 1e-5
    f.close()


@pytest.mark.parametrize("N,m,n,order,damping", [(24, 33, 131, "B_FIRST", 0.1), (12, 130, 67, "A_FIRST", 0.0)])
def test_odd_layer_with_objective_and_damped_loglik(gpu, N, m, n, order, damping):
    G = _samples(N, m, n)
    f = ffe.FlipFlop(G.to(gpu), order=order, damping=damping)
    ll = f.iterate(3)
    A, B = (F.double().cpu().numpy() for F in f.factors())
    psi = f.objective()
    f.close()
    ref = oracle.flipflop(G.numpy(), 3, order=order, damping=damping)
    assert oracle.kron_rel_error(A, B, ref.A, ref.B) < 1e-5
    assert abs(psi - oracle.objective(G.numpy(), A, B)) < 1e-5
    want = oracle.loglik(G.numpy(), A, B)
    assert abs(ll[-1] - want) < 1e-6 * abs(want)


# odd source rows (element loads), rows of whole 16-byte vectors, both
@pytest.mark.parametrize("m,n", [(131, 257), (264, 136), (129, 260)])
def test_packing_of_bf16_samples(gpu, m, n):
    G = _samples(20, m, n, torch.bfloat16).to(gpu)
    f = ffe.FlipFlop(G)
    got = {w: f.half_step(w).double() for w in "AB"}   # fixed factor I
    f.close()
    X = G.double()
    want = {"B": sum(x @ x.T for x in X) / (20 * n), "A": sum(x.T @ x for x in X) / (20 * m)}
    for w in "AB":   # products of exact bf16 values, fp32 sums over <= 5280 of them
        assert float((got[w] - want[w]).norm() / want[w].norm()) <= 1e-5


@pytest.mark.parametrize("dtype,T,m,n", [(torch.bfloat16, 1024, 256, 512), (torch.bfloat16, 1024, 256, 300),
                                         (torch.bfloat16, 1000, 256, 256), (torch.float32, 768, 64, 128)])
@pytest.mark.parametrize("order", ["B_FIRST", "A_FIRST"])
def test_tokens_in_place_and_identity_start(gpu, dtype, T, m, n, order):
    g = torch.Generator().manual_seed(11)
    x = (torch.randn(T, n, generator=g) * torch.arange(1, n + 1) ** -0.4).to(dtype)
    y = torch.randn(T, m, generator=g).to(dtype)
    xd, yd = x.to(gpu), y.to(gpu)
    out = []
    for start in ({}, {"A0": torch.eye(n, device=gpu), "B0": torch.eye(m, device=gpu)}):
        f = ffe.FlipFlop(tokens=(xd, yd), order=order, **start)
        f.iterate(2)
        out.append([F.double().cpu().numpy() for F in f.factors()])
        f.close()
    assert torch.equal(xd.cpu(), x) and torch.equal(yd.cpu(), y)
    # the explicit identity goes through a product with I, exact, and fp32
    # sums of squares where the identity start sums in fp64; on the bf16 path
    # a last bit of a weight moves roundings of weighted tokens
    lim = 1e-6 if dtype == torch.float32 else 1e-4
    assert oracle.kron_rel_error(*out[0], *out[1]) < lim
    ref = oracle.flipflop_tokens(x.double().numpy(), y.double().numpy(), 2) if order == "B_FIRST" else None
    if ref is not None:
        assert oracle.kron_rel_error(*out[0], ref.A, ref.B) < (1e-5 if dtype == torch.float32 else 5e-3)


def test_noalloc_at_its_scratch_limit(gpu):
    """477 x 477 with 11 fp32 samples fits the static scratch only without the
    padded factorisation rows: it runs as before, with the same results."""
    cfg = ffe.ff_config()
    cfg.m = cfg.n = 477
    cfg.N = 11
    assert ffe.ff_workspace_size(cfg) > ffe.FF_NOALLOC_SCRATCH_BYTES
    G = _samples(11, 477, 477).to(gpu)
    cfg.G = G.data_ptr()
    cfg.stream = torch.cuda.current_stream(gpu).cuda_stream
    cfg.damping = 0.1
    A = torch.empty(477, 477, device=gpu)
    B = torch.empty(477, 477, device=gpu)
    torch.cuda.synchronize()
    done, ll = ffe.ff_fit_noalloc(cfg, 2, A.data_ptr(), B.data_ptr())
    f = ffe.FlipFlop(G, damping=0.1)
    want = f.iterate(2)
    FA, FB = f.factors()
    f.close()
    assert done == 2 and np.allclose(ll, want, rtol=1e-12)
    assert torch.equal(A, FA) and torch.equal(B, FB)


@pytest.mark.parametrize("bad", ["A", "B", "AB"])
def test_which_factor_is_blamed(gpu, bad):
    """Both factorisations run side by side: the error names A if A is not
    positive definite, whichever failed first, and the handle stays usable."""
    m, n = 300, 150
    A, B = _spd(n, 1), _spd(m, 2)
    A2, B2 = A.clone(), B.clone()
    if "A" in bad:
        A2[140, 140] = -1.0
    if "B" in bad:
        B2[3, 3] = -1.0
    f = ffe.FlipFlop(_samples(4, m, n).to(gpu), A0=A2.to(gpu), B0=B2.to(gpu), damping=0.1)
    X = torch.randn(1, m, n, device=gpu)
    for call in (lambda: f.kron_apply(X, inverse=True), f.objective):
        with pytest.raises(ffe.FlipFlopError) as e:
            call()
        assert e.value.code == ffe.FF_ERR_NOT_SPD and f"factor {bad[0]} not positive" in str(e.value)
    psi = f.objective(A.to(gpu), B.to(gpu))
    want = oracle.objective(_samples(4, m, n).numpy(), A.double().numpy(), B.double().numpy())
    assert abs(psi - want) < 1e-5
    f.close()


@pytest.mark.parametrize("bad", ["A", "B", "AB"])
@pytest.mark.parametrize("m,n", [(300, 150), (64, 1000)])
def test_which_factor_the_quantiser_blames(gpu, bad, m, n):
    """As above for the quantiser's two factorisations, which run on the
    reversed factors: the pivot that fails first in time is B's."""
    A, B = _spd(n, 1), _spd(m, 2)
    A2, B2 = A.clone(), B.clone()
    if "A" in bad:
        A2[2, 2] = -1.0        # among the last pivots
    if "B" in bad:
        B2[m - 1, m - 1] = -1.0   # the first pivot
    f = ffe.FlipFlop(torch.zeros(1, m, n, device=gpu))
    W = torch.randn(m, n, generator=torch.Generator().manual_seed(3)).to(gpu)
    for _ in range(3):
        with pytest.raises(ffe.FlipFlopError) as e:
            f.quantize(W, A2.to(gpu), B2.to(gpu), gamma=2.0)
        assert e.value.code == ffe.FF_ERR_NOT_SPD
        assert f"factor {bad[0]} not positive definite in ff_quantize" in str(e.value)
    # and the handle stays usable
    _, _, alpha, beta, dist = f.quantize(W, A.to(gpu), B.to(gpu), gamma=2.0)
    assert torch.isfinite(alpha).all() and torch.isfinite(beta).all() and np.isfinite(dist)
    f.close()


@pytest.mark.parametrize("m,n", [(131, 257), (130, 256)])
def test_workspace_of_unpadded_factorisations(gpu, m, n):
    """A workspace without room for padded factorisation rows is taken, by the
    library and by the class, and gives the same results; less is refused."""
    G = _samples(20, m, n).to(gpu)
    full = ffe.FlipFlop.workspace_bytes(m, n, 20, "f32")

    def accepted(size):
        try:
            ffe.FlipFlop(G, workspace=torch.empty(size, dtype=torch.uint8, device=gpu)).close()
            return True
        except ValueError:
            return False
    # L and L^-1 of an odd width d, d x (d + 3) / 4 * 4 floats each, aligned to 256 bytes
    least = full
    for d in (m, n):
        pad = -(-d // 4) * 4
        least -= 2 * (-(-d * pad * 4 // 256) - -(-d * d * 4 // 256)) * 256
    assert least < full
    assert accepted(full) and accepted(least) and not accepted(least - 1) and not accepted(100)
    out = []
    for size in (full, least):
        f = ffe.FlipFlop(G, workspace=torch.empty(size, dtype=torch.uint8, device=gpu))
        ll = f.iterate(2)
        out.append((*f.factors(), ll))
        f.close()
    # the same steps on rows of other lengths: element loads in place of vectors
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]
