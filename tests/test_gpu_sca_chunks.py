"""The chunked strong-coupling kernels at the edges of their shapes against the
oracle: fewer slices than chunks, one more than a register chunk holds (8, 16
and 32 slices x 32 chunks; 16 and 32 x 16), the path that re-reads memory
(above 32 x 32 slices), columns that do not fill a workgroup, and the shape
for many columns.

Tolerances as for every strong-coupling application (element-wise, relative to
the largest output): complex128 1e-12, complex64 2e-5.
"""
import numpy as np
import pytest
import torch

from oracle import precond as pc
from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, to_host, rel_err, say, TAU, G

pytestmark = pytest.mark.gpu

TOL = {torch.complex128: 1e-12, torch.complex64: 2e-5}


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("dim,nx,ntau,nrhs", [
    (1, 2, 2, 1), (1, 2, 3, 3), (2, 4, 32, 1), (2, 6, 33, 2), (1, 6, 256, 1), (1, 6, 257, 2),
    (1, 10, 512, 1), (1, 10, 513, 1), (1, 4, 1024, 2), (1, 4, 1025, 1), (1, 2, 3000, 1),
    (3, 16, 20, 4), (3, 16, 257, 4),
])
def test_sca_chunks(dim, nx, ntau, nrhs, dtype):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    sigma = sigma_field(nx, ntau, 520, dim)
    x = gaussian_rhs(nx, ntau, range(521, 521 + nrhs), dim)
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    L = Lattice(nx, ntau, TAU, G, dtype, dim=dim)
    L.set_aux_field(to_dev(sigma))
    xd = to_dev(x, dtype)
    for alpha in (1.5, 2.0):
        say(f"sca chunks dim={dim} nx={nx} ntau={ntau} nrhs={nrhs} alpha={alpha} {dtype}")
        y = to_host(L.apply_precond(xd, Precond("sca", alpha=alpha), "Q"))
        D, Lb = pc.sca_setup(sigma, TAU, G, alpha)
        ref = np.stack([pc.sca_apply(v, D, Lb) for v in x])
        assert rel_err(y, ref) < TOL[dtype]
