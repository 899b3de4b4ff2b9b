"""Operators of dimension 1 and 2 through the kernel that holds a line of T per
thread: time extents around a wave's tile (64 slices in dimension 1, 64 / Nx in
dimension 2), both slices of Ntau = 2 at the antiperiodic boundary, several
right-hand sides, the scaled form (through Chebyshev) and the fused reductions
(through solves).

Tolerances as for every operator and preconditioner: 1e-13 / 1e-12 (complex128),
5e-6 / 2e-4 (complex64, Chebyshev), relative to the largest output; solves by the
oracle's residual, 10 tol.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import precond as pc
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, rel_err, say, TAU, G

pytestmark = pytest.mark.gpu


def _setup(dim, nx, ntau, nrhs, dtype):
    from paper_1008_3647_amd import Lattice
    sigma = sigma_field(nx, ntau, 850, dim)
    x = gaussian_rhs(nx, ntau, range(851, 851 + nrhs), dim)
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    L = Lattice(nx, ntau, TAU, G, dtype, dim=dim)
    L.set_aux_field(to_dev(sigma))
    return L, sigma, x, to_dev(x, dtype)


@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-13), (torch.complex64, 5e-6)])
@pytest.mark.parametrize("dim,nx,ntaus", [
    (1, 6, (2, 63, 129)), (1, 8, (64, 65)), (1, 10, (2, 64, 70)), (1, 12, (63, 66)),
    (1, 14, (65, 128)), (1, 16, (2, 64, 127)),
    (2, 8, (2, 7, 8, 17)), (2, 10, (6, 7)), (2, 12, (2, 5, 9)), (2, 14, (4, 11)),
    (2, 16, (2, 3, 4, 9)),
])
def test_operator_tiles(dim, nx, ntaus, dtype, tol):
    require_gpu()
    for ntau in ntaus:
        for nrhs in (1, 3):
            say(f"{dim}D lines nx={nx} ntau={ntau} rhs={nrhs} {dtype}")
            L, sigma, x, xd = _setup(dim, nx, ntau, nrhs, dtype)
            y, yd = to_host(L.apply_M(xd)), to_host(L.apply_Mdag(xd))
            for k in range(nrhs):
                assert rel_err(y[k], oracle.apply_M(x[k], sigma, TAU, G)) < tol
                assert rel_err(yd[k], oracle.apply_Mdag(x[k], sigma, TAU, G)) < tol


@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-12), (torch.complex64, 2e-4)])
@pytest.mark.parametrize("dim,nx,ntau", [(1, 10, 70), (2, 12, 7), (2, 8, 11)])
def test_scaled_form_and_reductions(dim, nx, ntau, dtype, tol):
    require_gpu()
    from paper_1008_3647_amd import Precond
    L, sigma, x, xd = _setup(dim, nx, ntau, 2, dtype)
    lam_max, eps = 7.0, 1e-2
    cheb = Precond("cheb", degree=8, eps=eps, lam_max=lam_max)
    y = to_host(L.apply_precond(xd, cheb, "Q"))
    for k in range(2):
        assert rel_err(y[k], pc.apply_cheb(x[k], sigma, TAU, G, 8, eps, lam_max)) < tol
    if dtype == torch.complex64:
        return
    stol = 1e-10

    def res(kind, z, k):
        r = oracle.apply_M(z, sigma, TAU, G)
        if kind == "Q":
            r = oracle.apply_Mdag(r, sigma, TAU, G)
        return np.linalg.norm(r - x[k]) / np.linalg.norm(x[k])

    wce = Precond("wce", wce_order=2)
    for kind, name, (z, st) in (
            ("Q", "cg", L.solve_cg_normal(xd, None, tol=stol)),
            ("Q", "cg cheb", L.solve_cg_normal(xd, cheb, tol=stol)),
            ("M", "bicgstab", L.solve_bicgstab(xd, "M", wce, tol=stol))):
        say(f"{dim}D {nx} x {ntau} {name} {st}")
        assert st["status"] == 0
        for k in range(2):
            assert res(kind, to_host(z)[k], k) < 10 * stol
