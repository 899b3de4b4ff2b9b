"""The force contraction on lattices with the block form of T at the sizes the
other tests leave out: every Nx / 2 odd (component boundary inside a wave), the
antiperiodic slice next to itself (Ntau = 2), several right-hand sides, and a
second field (cos sigma comes from the installed field).

Tolerances of the force tests: 1e-12 (complex128), 2e-5 (complex64), relative to
the largest entry."""
import numpy as np
import pytest
import torch

import oracle
from oracle import force as oforce
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, rel_err, say, TAU, G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-12), (torch.complex64, 2e-5)])
@pytest.mark.parametrize("nx,ntau,nrhs", [(6, 2, 1), (8, 3, 2), (10, 5, 3), (12, 2, 2), (14, 3, 1)])
def test_force_block(nx, ntau, nrhs, dtype, tol):
    require_gpu()
    from paper_1008_3647_amd import Lattice
    L = Lattice(nx, ntau, TAU, G, dtype)
    for seed in (830, 831):
        say(f"force {nx}^3 x {ntau} rhs={nrhs} {dtype} seed={seed}")
        sigma = sigma_field(nx, ntau, seed)
        X = gaussian_rhs(nx, ntau, range(840, 840 + nrhs))
        if dtype == torch.complex64:
            X = X.astype(np.complex64).astype(np.complex128)
        y = np.stack([oracle.apply_M(Xi, sigma, TAU, G) for Xi in X])
        if dtype == torch.complex64:
            y = y.astype(np.complex64).astype(np.complex128)
        L.set_aux_field(to_dev(sigma))
        g = to_host(L.force_dS_dsigma(to_dev(X, dtype), to_dev(y, dtype)))
        ref = sum(oforce.gradient(Xi, sigma, TAU, G) for Xi in X)
        assert rel_err(g, ref) < tol
