"""The preconditioned BiCGStab issues a check interval in pieces of a few
iterations and leaves out what is left of it once every right-hand side has
stopped (the flags come from pinned memory written by the solver's own
kernels). Nothing of that may show: solutions, iteration counts and counters
are those of whole intervals, also where the interval is shorter than a piece,
is no multiple of it, or is longer than the solve.
"""
import numpy as np
import pytest
import torch

import oracle
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, say, TAU, G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("check", [1, 2, 3, 5, 10, 64])
def test_interval_in_pieces(check):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    nx, ntau = 8, 24
    sigma = sigma_field(nx, ntau, 471)
    b = gaussian_rhs(nx, ntau, [472, 473, 474])
    b[2] = 0.0  # stops at once; the others run on
    L = Lattice(nx, ntau, TAU, G, torch.complex128)
    L.set_aux_field(to_dev(sigma))
    out = []
    for graph in (False, True, True):
        say(f"check_every={check} graph={graph}")
        x, st = L.solve_bicgstab(to_dev(b), "M", Precond("wce", wce_order=2), tol=1e-11,
                                 check_every=check, graph=graph)
        say(st)
        assert st["status"] == 0
        n = check * (-(-max(st["iters"]) // check))  # the check point that confirmed
        # two operators and two preconditioners an iteration, and order 2 holds
        # two operators and three M0^-1
        assert st["mv"] == n * (2 + 2 * 2) and st["m0inv"] == n * 2 * 3
        out.append((to_host(x), st))
    for x, st in out[1:]:
        assert np.array_equal(x, out[0][0])
        assert all(st[k] == out[0][1][k] for k in ("iters", "mv", "m0inv"))
    # one right-hand side alone, after a solve of three: the flags of the solve
    # before are not taken for this one's
    _, st1 = L.solve_bicgstab(to_dev(b[:1]), "M", Precond("wce", wce_order=2), tol=1e-11,
                              check_every=check)
    assert st1["status"] == 0 and st1["iters"][0] > 1


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("check", [1, 4, 7, 9, 64])
def test_fused_intervals(check, mixed):
    """The unpreconditioned form on a streaming lattice: it keeps whole intervals at
    every length. Converged (the oracle's residual), and FP64 counts whole intervals."""
    require_gpu()
    from paper_1008_3647_amd import Lattice
    nx, ntau, tol = 8, 24, 1e-10
    sigma = sigma_field(nx, ntau, 481)
    b = gaussian_rhs(nx, ntau, [482, 483])
    L = Lattice(nx, ntau, TAU, G, torch.complex128)
    L.set_aux_field(to_dev(sigma))
    for _ in range(2):
        say(f"fused check_every={check} mixed={mixed}")
        x, st = L.solve_bicgstab(to_dev(b), "M", tol=tol, mixed=mixed, check_every=check)
        say(st)
        assert st["status"] == 0
        if not mixed:
            assert st["mv"] == 2 * check * (-(-max(st["iters"]) // check))
        for k in range(2):
            r = oracle.apply_M(to_host(x)[k], sigma, TAU, G) - b[k]
            assert np.linalg.norm(r) <= 1.2 * tol * np.linalg.norm(b[k])
