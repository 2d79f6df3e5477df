"""Timed cases of the FlipFlop engine: what a user has it do, through its Python API.

A case names a `kind` of call and its sizes:

* ``fit``: one layer's whole job on samples that lie on the GPU: the handle,
  `iters` iterations, the factors (dense samples G, or tokens x, g);
* ``half``: one half step with a given fixed factor on a handle that is kept;
* ``apply`` / ``apply_inv``: the Kronecker product (or its inverse) of a
  handle's factors applied to a batch of matrices;
* ``objective``: the mismatch objective of given factors;
* ``quantise``: one WaterKron quantisation of a layer.

The listed cases run from the launch-bound 64 x 128 layer to the
8192 x 28672 one; `draw` gives others of the same ranges, odd sizes among
them.  Inputs are made on the GPU from the seed: samples with power-law
spectra on both sides, rotated, plus a low-rank term outside the Kronecker
model; factors with power-law spectra and a floor.
"""
import math

import torch

import paper_2609_14706_amd as ffe

DEV = "cuda:0"
P_IN, P_OUT = 1.2, 0.8   # decay of the input- and output-side spectra


def listed():
    return [
        # the smallest configuration: every step is a launch, nothing fills the GPU
        dict(name="fit_64x128_f32", kind="fit", m=64, n=128, N=256, dtype="f32", iters=20),
        # fp32 samples at a size no tile or vector divides, with the paper's damping
        dict(name="fit_1000x777_f32", kind="fit", m=1000, n=777, N=32, dtype="f32", iters=3, damping=0.1),
        # a small layer from few samples: two whitening passes, mostly factorisation
        dict(name="fit_768x512_bf16", kind="fit", m=768, n=512, N=16, dtype="bf16", iters=10),
        # odd sizes on the bf16 path (padded copies), the A-first order
        dict(name="fit_1500x2051_bf16", kind="fit", m=1500, n=2051, N=48, dtype="bf16", iters=3,
             order="A_FIRST"),
        # the headline layer, an attention projection at its full sample count (FlipFlop-2)
        dict(name="fit_4096x4096_bf16", kind="fit", m=4096, n=4096, N=128, dtype="bf16", iters=2),
        # an MLP down projection with heavy-tailed gradients (FlipFlop-1)
        dict(name="fit_4096x11008_bf16", kind="fit", m=4096, n=11008, N=64, dtype="bf16", iters=1,
             heavy=True),
        # the widest layer: one half step through its 28672 factor
        dict(name="half_8192x28672_bf16", kind="half", which="B", m=8192, n=28672, N=32, dtype="bf16"),
        # the per-token form at the paper's calibration size, 256 x 2048 tokens
        dict(name="tokens_4096x4096_bf16", kind="fit", m=4096, n=4096, T=524288, dtype="bf16", iters=1),
        # Table 1's Frobenius estimator: dense products with the factors themselves
        dict(name="frobenius_2048x2048_bf16", kind="fit", m=2048, n=2048, N=64, dtype="bf16", iters=2,
             damping=0.1, estimator="frobenius"),
        # Hessian-vector products with the estimate and with its inverse
        dict(name="apply_3000x2000", kind="apply", m=3000, n=2000, batch=8),
        dict(name="apply_inv_4096x4096", kind="apply_inv", m=4096, n=4096, batch=4),
        # the consumer of the factors: WaterKron at about two bits a weight.  Small on purpose:
        # on layers of 512 and more, one code that flips at a near tie (a last bit of a factor
        # decides it) changes about 2% of the codes after it, so that two correct results
        # cannot be compared entry by entry
        dict(name="quantise_160x128", kind="quantise", m=160, n=128, gamma=2.0),
    ]


def _size(rng, lo, hi):
    """Log-uniform in [lo, hi]; every other one a multiple of 64."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and v >= 64:
        v = v // 64 * 64
    return v


def draw(rng):
    kind = rng.choice(["fit_f32", "fit_bf16", "fit_bf16", "tokens", "half", "apply", "apply_inv",
                       "objective", "quantise"])
    if kind in ("fit_f32", "fit_bf16", "half", "objective"):
        bf16 = kind != "fit_f32"
        m, n = (_size(rng, 128, 6144), _size(rng, 128, 6144)) if bf16 else (_size(rng, 32, 1536),
                                                                           _size(rng, 32, 1536))
        most = (1 << 31 if bf16 else 1 << 27) // (m * n)
        least = min(most, 4 * -(-max(m, n) // min(m, n)))   # both factors determined
        N = max(1, min(512, int(math.exp(rng.uniform(math.log(max(least, 1)), math.log(max(most, least, 2)))))))
        c = dict(kind="fit" if kind.startswith("fit") else kind, m=m, n=n, N=N,
                 dtype="bf16" if bf16 else "f32")
        if kind == "half":
            c["which"] = rng.choice(["A", "B"])
        elif kind != "objective":
            c["iters"] = rng.randint(1, 3) if bf16 else rng.randint(2, 10)
            c["order"] = rng.choice(["A_FIRST", "B_FIRST"])
            if N * min(m, n) < 6 * max(m, n) or rng.random() < 0.3:
                c["damping"] = 0.1
        return c
    if kind == "tokens":
        m, n = _size(rng, 64, 4096), _size(rng, 64, 4096)
        est = rng.choice(["flipflop", "flipflop", "marginal", "input", "frobenius"])
        T = int(math.exp(rng.uniform(math.log(8 * max(m, n)), math.log(1 << 17))))
        dtype = rng.choice(["bf16", "bf16", "f32"])
        if dtype == "f32":
            m, n, T = max(32, m // 3), max(32, n // 3), T // 3
        c = dict(kind="fit", m=m, n=n, T=T, dtype=dtype, iters=rng.randint(1, 3), estimator=est)
        if est == "frobenius":
            c["damping"] = 0.1
        return c
    if kind == "quantise":
        return dict(kind="quantise", m=_size(rng, 40, 160), n=_size(rng, 40, 160), gamma=2.0)
    return dict(kind=kind, m=_size(rng, 64, 4096), n=_size(rng, 64, 4096), batch=rng.randint(1, 6))


# ------------------------------------------------------------------ inputs
def _gen(seed, *more):
    g = torch.Generator(device=DEV)
    g.manual_seed(hash((int(seed),) + more) & 0x7FFFFFFFFFFF)
    return g


def _spectrum(d, p):
    lam = torch.arange(1, d + 1, device=DEV, dtype=torch.float32) ** -p
    return lam * (d / lam.sum())


def _directions(d, count, g):
    u = torch.randn(count, d, device=DEV, generator=g)
    return u / u.norm(dim=1, keepdim=True)


def _factor(d, p, g, floor=0.01):
    """Dense SPD matrix: power-law spectrum plus a floor, rotated by reflections."""
    F = torch.diag(_spectrum(d, p) + floor)
    for u in _directions(d, 24, g):
        F -= torch.outer(F @ u, 2 * u)
        F -= torch.outer(2 * u, u @ F)
    return (F + F.T) / 2


def _noise(shape, g, heavy):
    z = torch.randn(shape, device=DEV, generator=g)
    if heavy:   # Student-t with four degrees of freedom, unit variance
        q = torch.zeros(shape, device=DEV)
        for _ in range(4):
            q += torch.randn(shape, device=DEV, generator=g) ** 2
        z *= (q / 4).rsqrt_() * (0.5 ** 0.5)
    return z


def _samples(c, seed):
    m, n, N = c["m"], c["n"], c["N"]
    g = _gen(seed, 1)
    sa, sb = _spectrum(n, P_IN).sqrt(), _spectrum(m, P_OUT).sqrt()
    ua, ub = _directions(n, 4, g), _directions(m, 4, g)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    G = torch.empty(N, m, n, dtype=dt, device=DEV)
    step = max(1, (1 << 27) // (m * n))
    r = 16
    for i in range(0, N, step):
        k = min(step, N - i)
        Z = _noise((k, m, n), g, c.get("heavy", False))
        Z *= sa
        Z *= sb[:, None]
        for u in ua:
            Z -= (Z.view(k * m, n) @ u).view(k, m, 1) * (2 * u)
        for u in ub:
            Z -= (2 * u)[:, None] * torch.matmul(u, Z).view(k, 1, n)
        for q in range(k):   # a tenth of the energy outside the Kronecker model
            U = torch.randn(m, r, device=DEV, generator=g) * (0.1 / r) ** 0.5
            Z[q].addmm_(U, torch.randn(r, n, device=DEV, generator=g))
        G[i:i + k] = Z
        del Z
    return G


def _tokens(c, seed):
    g = _gen(seed, 2)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    out = []
    for d, p, heavy in ((c["n"], P_IN, True), (c["m"], P_OUT, False)):
        s, us = _spectrum(d, p).sqrt(), _directions(d, 4, g)
        V = torch.empty(c["T"], d, dtype=dt, device=DEV)
        for i in range(0, c["T"], 65536):
            Z = _noise((min(65536, c["T"] - i), d), g, heavy) * s
            for u in us:
                Z -= (Z @ u)[:, None] * (2 * u)
            V[i:i + len(Z)] = Z
        out.append(V)
    return out   # x, g


def _factors(c, seed):
    return _factor(c["n"], P_IN, _gen(seed, 3)), _factor(c["m"], P_OUT, _gen(seed, 4))


def _options(c):
    return dict(order=c.get("order", "B_FIRST"), damping=c.get("damping", 0.0),
                estimator=c.get("estimator", "flipflop"))


def prepare(case, seed):
    c = case
    s = {"case": c}
    if c["kind"] == "fit":
        if "T" in c:
            s["src"] = {"tokens": tuple(_tokens(c, seed))}
        else:
            s["src"] = {"G": _samples(c, seed)}
        # the workspace is the program's: one for all its layers
        nbytes = ffe.FlipFlop.workspace_bytes(c["m"], c["n"], c.get("T", c.get("N")), c["dtype"], 0,
                                              rank1="T" in c)
        s["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    elif c["kind"] == "half":
        F = _factor(c["n"], P_IN, _gen(seed, 3)) if c["which"] == "B" else _factor(c["m"], P_OUT,
                                                                                   _gen(seed, 4))
        s.update(F=F, handle=ffe.FlipFlop(_samples(c, seed)))
    elif c["kind"] == "objective":
        A, B = _factors(c, seed)
        s.update(A=A, B=B, handle=ffe.FlipFlop(_samples(c, seed)))
    else:
        m, n = c["m"], c["n"]
        A, B = _factors(c, seed)
        # a handle that holds these factors (its one sample is not used)
        G = torch.zeros(1, m, n, device=DEV)
        s["handle"] = ffe.FlipFlop(G, A0=A, B0=B)
        g = _gen(seed, 5)
        if c["kind"] == "quantise":
            s["W"] = torch.randn(m, n, device=DEV, generator=g)
            s["workspace"] = torch.empty(ffe.FlipFlop.quantize_workspace_bytes(m, n), dtype=torch.uint8,
                                         device=DEV)
        else:
            s["X"] = torch.randn(c["batch"], m, n, device=DEV, generator=g)
    torch.cuda.synchronize()
    return s


def run(state):
    c = state["case"]
    if c["kind"] == "fit":
        f = ffe.FlipFlop(**state["src"], workspace=state["workspace"], **_options(c))
        loglik = f.iterate(c["iters"])
        A, B = f.factors()
        f.close()
        return {"A": A, "B": B, "loglik": loglik} if _options(c)["estimator"] == "flipflop" else {"A": A, "B": B}
    h = state["handle"]
    if c["kind"] == "half":
        return h.half_step(c["which"], state["F"])
    if c["kind"] == "objective":
        return h.objective(state["A"], state["B"])
    if c["kind"] == "quantise":
        Z, V, alpha, beta, dist = h.quantize(state["W"], gamma=c["gamma"], workspace=state["workspace"])
        return {"Z": Z, "V": V, "alpha": alpha, "beta": beta, "distortion": dist}
    return h.kron_apply(state["X"], inverse=c["kind"] == "apply_inv")


def work(case):
    """Each input read once and each output written once; the products as the
    method counts them (a triangular or symmetric product costs half a square
    one; a factorisation d^3 / 3)."""
    c = case
    m, n = float(c["m"]), float(c["n"])
    e = 2 if c.get("dtype") == "bf16" else 4
    if c["kind"] == "fit":
        iters, est = c["iters"], c.get("estimator", "flipflop")
        if "T" in c:
            T = float(c["T"])
            moment = T * (n * n + (m * m if est != "input" else 0))
            weights = {"flipflop": T * (n * n + m * m), "frobenius": 2 * T * (n * n + m * m)}.get(est, 0)
            one, inp = moment + weights, T * (m + n) * e
        else:
            N = float(c["N"])
            one, inp = N * m * n * (m + n) * (2 if est == "flipflop" else 3), N * m * n * e
        if est == "flipflop":
            one += (m ** 3 + n ** 3) / 3
        first = 0.0
        if "T" not in c:   # the first half step from the identity needs no whitening product
            d = n if c.get("order", "B_FIRST") == "B_FIRST" else m
            first = float(c["N"]) * m * n * d * (1 if est == "flipflop" else 2)
        return {"bytes": inp + 4 * (m * m + n * n), "flops": iters * one - first}
    if c["kind"] in ("half", "objective"):
        N = float(c["N"])
        both = c["kind"] == "objective"
        d, o = (n, m) if both or c["which"] == "B" else (m, n)   # fixed side, computed side
        fl = N * m * n * (m + n) + (d ** 3 + (o ** 3 if both else 0)) / 3
        return {"bytes": N * m * n * e + 4 * (d * d + o * o), "flops": fl}
    if c["kind"] == "quantise":
        return {"bytes": 4 * (m * m + n * n + 3 * m * n), "flops": m * m * n + m * n * n + (m ** 3 + n ** 3) / 3}
    b = float(c["batch"])
    fl = 2 * b * m * n * (m + n)
    if c["kind"] == "apply_inv":
        fl += (m ** 3 + n ** 3) / 3
    return {"bytes": 4 * (m * m + n * n + 2 * b * m * n), "flops": fl}


def tolerance(case):
    c = case
    if c["kind"] == "quantise":
        # a code whose quotient lies within the rounding of its fp32 sums from a tie may flip
        # (about one layer in a hundred of these sizes), and with it a few later ones
        return {"rel": 2e-3, "max": 0.99, "differ": 0.01}
    if c.get("dtype") == "bf16":
        return {"rel": 4e-3, "max": 0.2}
    if c["kind"] == "apply_inv":
        return {"rel": 1e-4, "max": 4e-3}
    return {"rel": 2e-5, "max": 1e-3}


# ------------------------------------------------------- the same in 64 bits
def _inv(F):
    return torch.cholesky_inverse(torch.linalg.cholesky(F))


def _moment(G, M, which):
    """(1/(N d)) sum_i G_i M G_i^T (which = "B") or of the G_i^T M G_i, d the size of M."""
    N = G.shape[0]
    out = 0
    for i in range(N):
        X = G[i].double() if which == "B" else G[i].double().T.contiguous()
        out = out + (X @ M) @ X.T.contiguous()
    out = out / (N * M.shape[0])
    return (out + out.T) / 2


def _weighted(U, V, M):
    """sum_t w_t u_t u_t^T / T with w_t = v_t^T M v_t (1 without M)."""
    T, out = U.shape[0], 0
    for i in range(0, T, 65536):
        u = U[i:i + 65536].double()
        if M is None:
            out = out + u.T.contiguous() @ u
        else:
            v = V[i:i + 65536].double()
            w = ((v @ M) * v).sum(1)
            out = out + (u * w[:, None]).T.contiguous() @ u
    return out / T


def _exact_fit(c, seed):
    m, n, est, kappa = c["m"], c["n"], c.get("estimator", "flipflop"), c.get("damping", 0.0)
    N = c.get("T", c.get("N"))
    if "T" in c:
        x, g = _tokens(c, seed)
    else:
        G = _samples(c, seed)
    F = {"A": torch.eye(n, device=DEV, dtype=torch.float64), "B": torch.eye(m, device=DEV, dtype=torch.float64)}
    order = "AB" if c.get("order", "B_FIRST") == "A_FIRST" or est in ("marginal", "input") else "BA"
    loglik = []
    for _ in range(c["iters"]):
        raw = None
        for s in order:
            o = "A" if s == "B" else "B"
            if est in ("marginal", "input"):
                new = torch.eye(m, device=DEV, dtype=torch.float64) if (s, est) == ("B", "input") else \
                    _weighted(g if s == "B" else x, None, None)
            else:
                M = F[o] if est == "frobenius" else _inv(F[o])
                if "T" in c:
                    new = _weighted(g, x, M) / n if s == "B" else _weighted(x, g, M) / m
                else:
                    new = _moment(G, M, s)
            raw = new
            d = new.shape[0]
            F[s] = new + kappa * (new.trace() / d) * torch.eye(d, device=DEV, dtype=torch.float64)
        if est == "flipflop":
            # sum_i tr(B^-1 G_i A^-1 G_i^T) = N d' tr(F^-1 F_undamped) for the factor updated last
            s = order[1]
            d_o = m if s == "A" else n
            tr = N * d_o * float((_inv(F[s]) * raw).sum())
            ld = {k: 2 * float(torch.linalg.cholesky(F[k]).diagonal().log().sum()) for k in "AB"}
            loglik.append(-0.5 * N * (m * ld["A"] + n * ld["B"]) - 0.5 * tr
                          - 0.5 * N * m * n * math.log(2 * math.pi))
        sc = F["A"].trace() / n
        F = {"A": F["A"] / sc, "B": F["B"] * sc}
    return dict(F, loglik=loglik) if est == "flipflop" else F


def _scales(M, gamma):
    """sqrt(gamma) |M|^(1/2d) / L_jj with L lower triangular and L^T L = M."""
    diag = torch.linalg.cholesky(M.flip(0, 1).contiguous()).diagonal().flip(0)
    return math.sqrt(gamma) * torch.exp(diag.log().mean()) / diag


def exact(case, seed):
    c = case
    if c["kind"] == "fit":
        return _exact_fit(c, seed)
    if c["kind"] == "half":
        if max(c["m"], c["n"]) > 12000:
            return None   # a 64-bit factorisation of the 28672 factor takes too long
        F = _factor(c["n"], P_IN, _gen(seed, 3)) if c["which"] == "B" else _factor(c["m"], P_OUT,
                                                                                   _gen(seed, 4))
        return _moment(_samples(c, seed), _inv(F.double()), c["which"])
    A, B = (F.double() for F in _factors(c, seed))
    if c["kind"] == "objective":
        M = _moment(_samples(c, seed), _inv(A), "B")
        ld = {k: 2 * float(torch.linalg.cholesky(F).diagonal().log().sum()) for k, F in (("A", A), ("B", B))}
        return math.log(float((_inv(B) * M).sum()) / c["m"]) + ld["A"] / c["n"] + ld["B"] / c["m"]
    if c["kind"] == "quantise":   # codes of near ties may differ, and all that follows from them
        return {"Z": None, "V": None, "alpha": _scales(A, c["gamma"]), "beta": _scales(B, c["gamma"]),
                "distortion": None}
    X = torch.randn(c["batch"], c["m"], c["n"], device=DEV, generator=_gen(seed, 5)).double()
    if c["kind"] == "apply_inv":
        A, B = _inv(A), _inv(B)
    return torch.stack([B @ x @ A for x in X])
