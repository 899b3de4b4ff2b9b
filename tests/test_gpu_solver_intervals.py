"""The unfused BiCGStab without a preconditioner (Nx = 4, dimensions 1 and 2), whose
check intervals are issued in pieces of ten iterations, at intervals below, at and
above that length: solutions and counters are those of whole intervals, from a graph
and launch by launch. And the early end of a long interval, by its cost: a solve of
a few tens or hundreds of iterations checked every 2000 must not launch the others.
"""
import time

import numpy as np
import pytest
import torch

import oracle
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, say, TAU, G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("check", [1, 7, 10, 11, 20, 25, 64])
@pytest.mark.parametrize("dim,nx", [(3, 4), (1, 8), (2, 6), (2, 8)])
def test_unpreconditioned_intervals(dim, nx, check):
    require_gpu()
    from paper_1008_3647_amd import Lattice
    ntau, tol = 20, 1e-9
    sigma = sigma_field(nx, ntau, 491, dim)
    b = gaussian_rhs(nx, ntau, [492, 493, 494], dim)
    b[1] = 0.0  # stops at once
    L = Lattice(nx, ntau, TAU, G, torch.complex128, dim=dim)
    L.set_aux_field(to_dev(sigma))
    bd = to_dev(b)
    out = []
    for graph in (False, True, True):
        say(f"dim={dim} nx={nx} check_every={check} graph={graph}")
        x, st = L.solve_bicgstab(bd, "M", tol=tol, check_every=check, graph=graph)
        say(st)
        assert st["status"] == 0
        assert st["mv"] == 2 * check * (-(-max(st["iters"]) // check))
        r = to_host(L.apply_M(x)) - b
        for k in range(3):
            assert np.linalg.norm(r[k]) <= 1.2 * tol * np.linalg.norm(b[k])
        out.append((to_host(x), st))
    for x, st in out[1:]:
        assert np.array_equal(x, out[0][0])
        assert all(st[k] == out[0][1][k] for k in ("iters", "mv"))


@pytest.mark.parametrize("dim,nx,precond", [(3, 8, "wce"), (3, 4, "wce"), (2, 8, "none")])
def test_long_interval_ends_early(dim, nx, precond):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    ntau = 12
    L = Lattice(nx, ntau, TAU, G, torch.complex128, dim=dim)
    L.set_aux_field(to_dev(0.3 * sigma_field(nx, ntau, 495, dim)))
    bd = to_dev(gaussian_rhs(nx, ntau, [496], dim))
    p = Precond("wce", wce_order=2) if precond == "wce" else None

    def best(check):
        runs = []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            _, st = L.solve_bicgstab(bd, "M", p, tol=1e-8, check_every=check, maxit=10000)
            runs.append(time.perf_counter() - t)
            assert st["status"] == 0 and max(st["iters"]) < 300
        return min(runs), max(st["iters"])

    (short, n), (long, m) = best(10), best(2000)
    say(f"dim={dim} nx={nx} {precond}: {n} iterations, checked every 10 {1e3 * short:.2f} ms, "
        f"every 2000 ({m} iterations) {1e3 * long:.2f} ms")
    # 2000 iterations of launches that do nothing take 50 ms and more
    assert long < 4 * short + 5e-3
