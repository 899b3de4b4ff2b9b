"""Order-0 weak-coupling applications on Nx = 16 with one slice a workgroup, where the
scan turns the modes into (1 - lam Z)^{-1} of them in place: time extents of 2 and
more, both sides of the rules that choose it (complex128 up to 600 slices in all,
complex64 from 513 to 600), and inactive right-hand sides in a solve.

Tolerances as for every weak-coupling application (element-wise, relative to
the largest output): complex128 1e-12, complex64 2e-5.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import precond as pc
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, rel_err, say, TAU, G

pytestmark = pytest.mark.gpu

TOL = {torch.complex128: 1e-12, torch.complex64: 2e-5}


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("ntau,nrhs", [(2, 1), (3, 3), (9, 2), (129, 1), (512, 1), (513, 1),
                                       (600, 1), (601, 1)])
def test_order_0(ntau, nrhs, dtype):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    nx = 16
    sigma = sigma_field(nx, ntau, 690)
    x = gaussian_rhs(nx, ntau, range(691, 691 + nrhs))
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    L = Lattice(nx, ntau, TAU, G, dtype)
    L.set_aux_field(to_dev(sigma))
    for euler in (False, True):
        p = Precond("wce", wce_order=0, euler=euler)
        for op, ref in (("M", pc.wce_apply), ("Mdag", pc.wce_apply_dag)):
            say(f"wce order 0 ntau={ntau} nrhs={nrhs} euler={euler} {op} {dtype}")
            y = to_host(L.apply_precond(to_dev(x, dtype), p, op))
            for k in range(nrhs):
                assert rel_err(y[k], ref(x[k], sigma, TAU, G, 0)) < TOL[dtype]


def test_order_0_inactive_rhs():
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    nx, ntau, tol = 16, 6, 1e-10
    sigma = sigma_field(nx, ntau, 695)
    b = gaussian_rhs(nx, ntau, [696, 697, 698])
    b[1] = 0.0
    L = Lattice(nx, ntau, TAU, G, torch.complex128)
    L.set_aux_field(to_dev(sigma))
    x, st = L.solve_bicgstab(to_dev(b), "M", Precond("wce", wce_order=0), tol=tol)
    x = to_host(x)
    say(st)
    assert st["status"] == 0 and np.all(x[1] == 0)
    for k in (0, 2):
        r = oracle.apply_M(x[k], sigma, TAU, G) - b[k]
        assert np.linalg.norm(r) <= 1.2 * tol * np.linalg.norm(b[k])
