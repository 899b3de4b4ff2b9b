"""The one-launch M^T M of the Chebyshev factors against the oracle: time
extents of 2 and 3 (every neighbour wraps), extents that leave a short last
workgroup, an odd number of factors and an even one (the vectors alternate),
and both sides of the rules that choose the slices per workgroup (Nx = 6, 8:
2048 slices in all, Nx = 10, 12: 512, complex64 Nx = 14: 1024) or two launches
(complex128 Nx = 14 above 512).

Tolerances as for every Chebyshev application: complex128 1e-12, complex64 2e-4.
"""
import numpy as np
import pytest
import torch

from oracle import precond as pc
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, rel_err, say, TAU, G

pytestmark = pytest.mark.gpu

TOL = {torch.complex128: 1e-12, torch.complex64: 2e-4}


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("nx,ntau,nrhs", [
    (8, 2, 1), (8, 3, 2), (8, 10, 3), (8, 2049, 1), (12, 2, 1), (12, 7, 3), (12, 514, 1), (12, 259, 1), (12, 44, 6),
    (16, 2, 2), (16, 5, 1), (6, 2, 1), (6, 9, 2), (6, 2050, 1), (10, 4, 2), (10, 514, 1),
    (14, 3, 2), (14, 513, 1), (14, 1026, 1),
])
def test_chebyshev_fused(nx, ntau, nrhs, dtype):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    sigma = sigma_field(nx, ntau, 730)
    x = gaussian_rhs(nx, ntau, range(731, 731 + nrhs))
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    L = Lattice(nx, ntau, TAU, G, dtype)
    L.set_aux_field(to_dev(sigma))
    for degree in (1, 2, 4):
        say(f"cheb fused nx={nx} ntau={ntau} nrhs={nrhs} degree={degree} {dtype}")
        p = Precond("cheb", degree=degree, eps=1e-2, lam_max=7.0)
        y = to_host(L.apply_precond(to_dev(x, dtype), p, "Q"))
        ref = np.stack([pc.apply_cheb(v, sigma, TAU, G, degree, 1e-2, 7.0) for v in x])
        assert rel_err(y, ref) < TOL[dtype]
