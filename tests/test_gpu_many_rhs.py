"""More right-hand sides than one dimension of a launch grid holds (65,535, two
components each): the weak-coupling application on the smallest lattice of its fused
launches. The right-hand sides repeat, so the first few are compared with the
oracle and every other one bit for bit with its first occurrence.

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
def test_wce_many_rhs(dtype):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    nx, ntau, few, times = 6, 2, 5, 6556
    nrhs = few * times  # 32,780
    sigma = sigma_field(nx, ntau, 620)
    x = gaussian_rhs(nx, ntau, range(621, 621 + few))
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    L = Lattice(nx, ntau, TAU, G, dtype)
    L.set_aux_field(to_dev(sigma))
    xd = to_dev(x, dtype).repeat(times, 1, 1, 1, 1)
    for op, ref in (("M", pc.wce_apply), ("Mdag", pc.wce_apply_dag)):
        say(f"wce {nrhs} rhs {op} {dtype}")
        y = L.apply_precond(xd, Precond("wce", wce_order=1), op)
        for k in range(few):
            assert rel_err(to_host(y[k]), ref(x[k], sigma, TAU, G, 1)) < TOL[dtype]
        y = y.reshape((times, few) + y.shape[1:])
        assert bool((y == y[:1]).all())
