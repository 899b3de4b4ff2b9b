"""The fused weak-coupling launches at every shape of their slab split against
the oracle: slabs of 1, of lengths that leave a short last slab, of the whole
time extent, and scans whose chunks of slabs exceed what a thread keeps in
registers (8 slabs times 8 chunks, or 16 times 16).

Tolerances as for every weak-coupling application (element-wise, relative to
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
@pytest.mark.parametrize("nx,ntau,nrhs,slabs", [
    (8, 7, 3, (1, 2, 3, 7)), (12, 6, 1, (1, 4, 6)), (16, 9, 2, (1, 2, 4, 8, 9)), (8, 2, 1, (1, 2)),
    (6, 7, 2, (1, 2, 3, 7)), (10, 5, 3, (1, 2, 5)), (14, 5, 1, (1, 3)),
    (16, 150, 2, (1,)),   # 32-column scan, more than 8 x 8 slabs
    (8, 600, 1, (1,)),    # 16-column scan, more than 16 x 16 slabs
])
def test_wce_slabs(nx, ntau, nrhs, slabs, dtype):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    sigma = sigma_field(nx, ntau, 660)
    x = gaussian_rhs(nx, ntau, range(661, 661 + nrhs))
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    L = Lattice(nx, ntau, TAU, G, dtype)
    L.set_aux_field(to_dev(sigma))
    xd = to_dev(x, dtype)
    for order in (0, 2):
        p = Precond("wce", wce_order=order)
        refs = {"M": np.stack([pc.wce_apply(v, sigma, TAU, G, order) for v in x]),
                "Mdag": np.stack([pc.wce_apply_dag(v, sigma, TAU, G, order) for v in x])}
        for slab in (0,) + slabs:  # 0: the default rule
            L.tune(slab=slab)
            for op, ref in refs.items():
                say(f"wce slabs nx={nx} ntau={ntau} d={order} slab={slab} {op} {dtype}")
                assert rel_err(to_host(L.apply_precond(xd, p, op)), ref) < TOL[dtype]
