"""Workloads of the library's public entry points, for timing and for comparing
outputs between two versions of the code.

`listed()` names the workloads, `draw(rng)` gives one more of the same ranges,
`prepare` builds what a program holds before the call, `run` makes one pass,
`work` states the least traffic and arithmetic of a pass, and `exact` computes
the same outputs with plain torch in complex128, by Fourier transforms.

Physics throughout: tau = 0.05, g = 5 (the unitary point of the paper), sigma iid
uniform on [-pi, pi], complex vectors with Re, Im iid N(0, 1/2).
"""
from __future__ import annotations

import cmath
import math

import torch

from paper_1008_3647_amd import Lattice, Precond

TAU, G = 0.05, 5.0
A = math.sqrt(2.0) * math.sqrt(math.exp(TAU * G) - 1.0)
DTYPES = {"c64": torch.complex64, "c128": torch.complex128}
# sites x right-hand sides of the largest listed operator call: nothing drawn exceeds it
MOST = 16 ** 3 * 800 * 8


def listed():
    return [
        # the smallest call: one operator application on the lattice of the HMC
        # thermalization chain and of the paper's smallest sweeps (general slice kernel)
        dict(name="op_M_6x50", kind="op", dim=3, nx=6, ntau=50, nrhs=1, dtype="c128", op="M"),
        # the paper's sweep lattices that are not multiples of 4, odd time extent, a
        # few right-hand sides
        dict(name="op_Mdag_10x201_r3", kind="op", dim=3, nx=10, ntau=201, nrhs=3, dtype="c128",
             op="Mdag"),
        # the operator inside every FP32-refined solve at the benchmark's size
        dict(name="op_M_16x400_r8_c64", kind="op", dim=3, nx=16, ntau=400, nrhs=8, dtype="c64",
             op="M"),
        # the largest call: the FP64 operator on twice the benchmark's time extent
        dict(name="op_Mdag_16x800_r8", kind="op", dim=3, nx=16, ntau=800, nrhs=8, dtype="c128",
             op="Mdag"),
        # lattices of lower dimension
        dict(name="op_M_2d_16x1000_r8", kind="op", dim=2, nx=16, ntau=1000, nrhs=8, dtype="c128",
             op="M"),
        # the weak-coupling preconditioner inside the FP32-refined solve
        dict(name="wce2_M_16x400_r8_c64", kind="precond", pc="wce", order=2, euler=False, nx=16,
             ntau=400, nrhs=8, dtype="c64", op="M"),
        # the same with Euler weights, transposed, as an HMC force applies it
        dict(name="wce2e_Mdag_12x200", kind="precond", pc="wce", order=2, euler=True, nx=12,
             ntau=200, nrhs=1, dtype="c128", op="Mdag"),
        # the Chebyshev preconditioner of CG on the preconditioner grid's lattice
        dict(name="cheb16_Q_8x160_r4", kind="precond", pc="cheb", degree=16, eps=1e-3, nx=8,
             ntau=160, nrhs=4, dtype="c128", op="Q"),
        # the strong-coupling preconditioner of CG on the same lattice
        dict(name="sca_Q_8x160_r4", kind="precond", pc="sca", alpha=2.0, nx=8, ntau=160, nrhs=4,
             dtype="c128", op="Q"),
        # what a molecular-dynamics step does besides its two solves: install the new
        # field, contract the force
        dict(name="field_force_12x200", kind="force", nx=12, ntau=200, nrhs=1, dtype="c128"),
        # molecular dynamics, solves included
        dict(name="hmc_12x200", kind="hmc", nx=12, ntau=200, nsteps=2),
        # the flagship: FP32-refined two-step BiCGStab at the benchmark's check interval, to
        # the paper's tolerance
        dict(name="solve_16x400_r8", kind="solve", nx=16, ntau=400, nrhs=8, pc="none"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["op", "op", "op", "precond", "precond", "precond", "force", "hmc", "solve"])
    dtype = rng.choice(["c64", "c128"])
    if kind == "op":
        dim = rng.choice([1, 2, 3, 3, 3, 3])
        nx = rng.choice([4, 6, 8, 10, 12, 14, 16])
        ntau = _log_int(rng, 40, 800) if dim == 3 else _log_int(rng, 500, 16000)
        nrhs = rng.randint(1, 8) if dim == 3 else _log_int(rng, 1, 64)
        return dict(kind=kind, dim=dim, nx=nx, ntau=ntau,
                    nrhs=max(1, min(nrhs, MOST // (nx ** dim * ntau))), dtype=dtype,
                    op=rng.choice(["M", "Mdag"]))
    if kind == "precond":
        pc = rng.choice(["wce", "wce", "cheb", "sca"])
        base = dict(kind=kind, pc=pc, nx=rng.choice([6, 8, 10, 12, 16]),
                    ntau=_log_int(rng, 50, 400), nrhs=rng.randint(1, 8), dtype=dtype)
        if pc == "wce":
            return dict(base, order=rng.randint(0, 4), euler=rng.random() < 0.5,
                        op=rng.choice(["M", "Mdag"]))
        if pc == "cheb":
            return dict(base, degree=rng.choice([8, 16]), eps=rng.choice([1e-2, 1e-3]), op="Q")
        return dict(base, alpha=rng.choice([1.5, 2.0, 3.0]), op="Q")
    if kind == "force":
        return dict(kind=kind, nx=rng.choice([6, 8, 10, 12, 16]), ntau=_log_int(rng, 50, 400),
                    nrhs=rng.randint(1, 4), dtype=dtype)
    if kind == "hmc":
        return dict(kind=kind, nx=rng.choice([6, 8, 10, 12]), ntau=_log_int(rng, 50, 200),
                    nsteps=rng.randint(1, 3))
    return dict(kind=kind, nx=rng.choice([8, 10, 12, 16]), ntau=_log_int(rng, 80, 240),
                nrhs=rng.randint(1, 6), pc=rng.choice(["none", "wce"]))


# ---------------------------------------------------------------------------
# inputs


def _shape(case):
    return (case["ntau"],) + (case["nx"],) * case.get("dim", 3)


def _inputs(case, seed):
    """sigma and the named vectors of a case, in 64 bits, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = _shape(case)
    kw = dict(generator=gen, device="cuda", dtype=torch.float64)
    sigma = (2.0 * torch.rand(shape, **kw) - 1.0) * math.pi

    def vectors(n):
        re, im = torch.randn((n,) + shape, **kw), torch.randn((n,) + shape, **kw)
        return torch.complex(re, im) * math.sqrt(0.5)

    kind = case["kind"]
    if kind in ("op", "precond"):
        return dict(sigma=sigma, x=vectors(case["nrhs"]).to(DTYPES[case["dtype"]]))
    if kind == "force":
        dt = DTYPES[case["dtype"]]
        return dict(sigma=sigma, X=vectors(case["nrhs"]).to(dt), y=vectors(case["nrhs"]).to(dt))
    if kind == "hmc":
        return dict(sigma=sigma, pi=torch.randn(shape, **kw), eta=vectors(1))
    return dict(sigma=sigma, b=vectors(case["nrhs"]))


def _precond(case):
    pc = case["pc"]
    if pc == "wce":
        return Precond("wce", wce_order=case.get("order", 2), euler=case.get("euler", False))
    if pc == "cheb":
        return Precond("cheb", degree=case["degree"], eps=case["eps"])
    if pc == "sca":
        return Precond("sca", alpha=case["alpha"])
    return None


def prepare(case, seed):
    state = dict(_inputs(case, seed), case=case)
    lat = Lattice(case["nx"], case["ntau"], TAU, G, DTYPES[case.get("dtype", "c128")],
                  dim=case.get("dim", 3))
    lat.set_aux_field(state["sigma"])
    state["lattice"] = lat
    if case["kind"] in ("precond", "solve"):
        state["precond"] = _precond(case)
    if case["kind"] == "hmc":
        state["precond"] = Precond("wce", wce_order=2, euler=True)
        state["phi"] = lat.apply_Mdag(state["eta"])
    return state


def run(state):
    case, lat = state["case"], state["lattice"]
    kind = case["kind"]
    if kind == "op":
        return lat.apply_M(state["x"]) if case["op"] == "M" else lat.apply_Mdag(state["x"])
    if kind == "precond":
        return lat.apply_precond(state["x"], state["precond"], op=case["op"])
    if kind == "force":
        lat.set_aux_field(state["sigma"])
        return lat.force_dS_dsigma(state["X"], state["y"])
    if kind == "hmc":
        sigma, pi, actions, _ = lat.hmc_leapfrog(state["sigma"], state["pi"], state["phi"], 0.0025,
                                                 case["nsteps"], state["precond"], tol=1e-12)
        return {"sigma": sigma, "pi": pi, "actions": actions}
    x, _ = lat.solve_bicgstab(state["b"], "two_step", state["precond"], tol=1e-12, mixed=True,
                              check_every=60)
    return x


def work(case):
    """Least traffic (inputs read once, outputs written once) and arithmetic (one
    kinetic factor per axis and slice, in its block form of about nx / 4 real
    multiply-adds per complex value; a solve: those of one operator call)."""
    dim = case.get("dim", 3)
    sites = case["nx"] ** dim * case["ntau"]
    nrhs = case.get("nrhs", 1)
    c = 8 if case.get("dtype", "c128") == "c64" else 16
    op = sites * nrhs * (dim * (case["nx"] + 8) + 4)
    kind = case["kind"]
    if kind == "op":
        return {"bytes": sites * (2 * c * nrhs + c // 2), "flops": op}
    if kind == "precond":
        times = {"wce": 2 * (case.get("order", 0) + 1), "cheb": 2 * case.get("degree", 0),
                 "sca": 1}[case["pc"]]
        flops = op * times if case["pc"] != "sca" else 20 * sites * nrhs
        return {"bytes": sites * (2 * c * nrhs + c // 2), "flops": flops}
    if kind == "force":
        return {"bytes": sites * (2 * c * nrhs + 16), "flops": op}
    if kind == "hmc":
        return {"bytes": sites * (4 * 8 + 16), "flops": op * 2 * (case["nsteps"] + 1)}
    return {"bytes": sites * (2 * 16 * nrhs + 8), "flops": 2 * op}


# ---------------------------------------------------------------------------
# the same in plain torch, complex128


def _kinetic(nx, dim):
    k = 2.0 * math.pi * torch.fft.fftfreq(nx, dtype=torch.float64, device="cuda")
    e = torch.zeros((nx,) * dim, dtype=torch.float64, device="cuda")
    for a in range(dim):
        e = e + (0.5 * k ** 2).reshape((nx,) + (1,) * (dim - 1 - a))
    return torch.exp(-TAU * e)


def _exp_k(v, dim):
    axes = tuple(range(-dim, 0))
    return torch.fft.ifftn(torch.fft.fftn(v, dim=axes) * _kinetic(v.shape[-1], dim), dim=axes)


def _sign(ntau, dim):
    s = torch.full((ntau,), -1.0, dtype=torch.float64, device="cuda")
    s[-1] = 1.0
    return s.reshape((ntau,) + (1,) * dim)


def _hop(v, f, dim):
    """The off-diagonal part of M with the field factor f: slice t to slice t + 1."""
    return torch.roll(_sign(v.shape[1], dim) * _exp_k(f * v, dim), 1, dims=1)


def _hop_dag(v, f, dim):
    return _sign(v.shape[1], dim) * f * _exp_k(torch.roll(v, -1, dims=1), dim)


def _m(v, sigma):
    return v + _hop(v, 1.0 + A * torch.sin(sigma), sigma.dim() - 1)


def _mdag(v, sigma):
    return v + _hop_dag(v, 1.0 + A * torch.sin(sigma), sigma.dim() - 1)


def _m0_inv(v, adjoint):
    """Inverse of M at A = 0: diagonal in momentum and antiperiodic frequency."""
    ntau, nx = v.shape[1], v.shape[-1]
    t = torch.arange(ntau, dtype=torch.float64, device="cuda").reshape(ntau, 1, 1, 1)
    twist = torch.exp(-1j * math.pi * t / ntau)
    w = 2.0 * math.pi * torch.fft.fftfreq(ntau, dtype=torch.float64, device="cuda") + math.pi / ntau
    symbol = 1.0 - torch.exp(-1j * w).reshape(ntau, 1, 1, 1) * _kinetic(nx, 3)
    symbol = symbol.conj() if adjoint else symbol
    axes = (1, 2, 3, 4)
    return torch.fft.ifftn(torch.fft.fftn(v * twist, dim=axes) / symbol, dim=axes) / twist


def _wce(v, sigma, order, weights, adjoint):
    s = torch.sin(sigma)
    total = torch.zeros_like(v)
    term = v if adjoint else _m0_inv(v, False)
    for m in range(order + 1):
        total = total + weights[m] * term
        if m < order:
            if adjoint:
                term = -A * _hop_dag(_m0_inv(term, True), s, 3)
            else:
                term = -A * _m0_inv(_hop(term, s, 3), False)
    return _m0_inv(total, True) if adjoint else total


def _cheb(v, sigma, degree, eps):
    h = 0.5 * (1.0 + eps)
    th = [2.0 * math.pi * k / (degree + 1) for k in range(1, degree + 1)]
    roots = [complex(h * (1.0 - math.cos(a)), -math.sqrt(eps) * math.sin(a)) for a in th]
    inverse = h
    for z in roots:
        inverse *= h - z
    factor = cmath.exp(-cmath.log(inverse) / degree)
    lam = (1.0 + float((1.0 + A * torch.sin(sigma)).abs().max())) ** 2
    for z in sorted(roots, key=lambda r: (r.real * 7.3) % 1.0):  # spread out: smooth growth
        v = factor * (_mdag(_m(v, sigma), sigma) / lam - z * v)
    return v


def _sca(v, sigma, alpha):
    b = 1.0 + A * torch.sin(sigma)
    n = b.shape[0]
    d = [alpha + b[0] ** 2]
    for t in range(1, n):
        d.append(alpha + b[t] ** 2 - b[t - 1] ** 2 / d[t - 1])
    d[n - 1] = d[n - 1] - b[n - 1] ** 2 / d[0]
    low = [b[t] / d[t] for t in range(n - 1)] + [b[n - 1] / d[0]]
    w = [v[:, 0]]
    for t in range(1, n):
        w.append(v[:, t] + low[t - 1] * w[t - 1])
    w[n - 1] = w[n - 1] - low[n - 1] * w[0]
    x = [w[t] / d[t] for t in range(n)]
    for t in range(n - 2, -1, -1):
        x[t] = x[t] + low[t] * x[t + 1]
    x[0] = x[0] - low[n - 1] * x[n - 1]
    return torch.stack(x, dim=1)


def _force(X, y, sigma):
    ty = _exp_k(torch.roll(y, -1, dims=1), 3)
    return -2.0 * A * torch.cos(sigma) * _sign(sigma.shape[0], 3) * (X * ty.conj()).real.sum(0)


def _solve(b, sigma, adjoint):
    """M x = b (adjoint: M^T x = b) for one vector: BiCGStab behind a weak-coupling
    preconditioner, repeated on the residual until that is at rounding level."""
    op = _mdag if adjoint else _m
    x, r = torch.zeros_like(b), b
    for _ in range(4):
        d, rr, shadow = torch.zeros_like(b), r, r
        rho, alpha, omega = 1.0, 1.0, 1.0
        p, v = torch.zeros_like(b), torch.zeros_like(b)
        for _ in range(80):
            rho, last = torch.sum(shadow.conj() * rr), rho
            p = rr + (rho / last) * (alpha / omega) * (p - omega * v)
            ph = _wce(p, sigma, 2, (1.0, 1.0, 1.0), adjoint)
            v = op(ph, sigma)
            alpha = rho / torch.sum(shadow.conj() * v)
            s = rr - alpha * v
            sh = _wce(s, sigma, 2, (1.0, 1.0, 1.0), adjoint)
            t = op(sh, sigma)
            omega = torch.sum(t.conj() * s) / torch.sum(t.conj() * t)
            d = d + alpha * ph + omega * sh
            rr = s - omega * t
            if float(torch.linalg.vector_norm(rr)) < 1e-8 * float(torch.linalg.vector_norm(r)):
                break
        x = x + d
        r = b - op(x, sigma)
        if float(torch.linalg.vector_norm(r)) < 4e-15 * float(torch.linalg.vector_norm(b)):
            break
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        return None  # minutes in plain torch
    i = _inputs(case, seed)
    sigma = i["sigma"]
    if kind == "op":
        return (_m if case["op"] == "M" else _mdag)(i["x"].to(torch.complex128), sigma)
    if kind == "precond":
        x = i["x"].to(torch.complex128)
        if case["pc"] == "wce":
            d = case["order"]
            weights = [1.0] * (d + 1)
            if case["euler"]:  # of the partial sums, binomial at p = 1/2
                weights = [sum(math.comb(d, k) for k in range(m, d + 1)) / 2.0 ** d
                           for m in range(d + 1)]
            return _wce(x, sigma, d, weights, case["op"] == "Mdag")
        if case["pc"] == "cheb":
            return _cheb(x, sigma, case["degree"], case["eps"])
        return _sca(x, sigma, case["alpha"])
    if kind == "force":
        return _force(i["X"].to(torch.complex128), i["y"].to(torch.complex128), sigma)
    pi, phi, dt, n = i["pi"], _mdag(i["eta"], sigma), 0.0025, case["nsteps"]
    actions = []
    for step in range(n + 1):
        y = _solve(phi, sigma, True)
        actions.append(float(torch.sum(y.abs() ** 2)))
        grad = _force(_solve(y, sigma, False), y, sigma)
        pi = pi - (0.5 * dt if step in (0, n) else dt) * grad
        if step < n:
            sigma = sigma + dt * pi
    return {"sigma": sigma, "pi": pi, "actions": actions}
