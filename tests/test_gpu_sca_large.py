"""Strong-coupling applications on vectors of 4 GiB and more, which leave the 32-bit
offsets of the register form: a few right-hand sides against the same ones alone
(the register form, checked against the oracle elsewhere).

Tolerances as for every strong-coupling application: complex128 1e-12, complex64 2e-5.
"""
import pytest
import torch

from synthetic import sigma_field
from gpu_util import require_gpu, to_dev, say, TAU, G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,nrhs,tol", [(torch.complex128, 165, 1e-12),
                                            (torch.complex64, 330, 2e-5)])
def test_sca_beyond_4gib(dtype, nrhs, tol):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    nx, ntau = 16, 400
    L = Lattice(nx, ntau, TAU, G, dtype)
    L.set_aux_field(to_dev(sigma_field(nx, ntau, 530)))
    gen = torch.Generator(device="cuda").manual_seed(531)
    x = torch.randn((nrhs,) + L.shape, generator=gen, dtype=dtype, device="cuda")
    assert x.nbytes >= 2 ** 32
    p = Precond("sca", alpha=2.0)
    y = L.apply_precond(x, p, "Q")
    for k in (0, nrhs // 2, nrhs - 1):
        say(f"sca of {x.nbytes >> 20} MiB, rhs {k}, {dtype}")
        one = L.apply_precond(x[k:k + 1].clone(), p, "Q")[0]
        assert float((y[k] - one).abs().max() / one.abs().max()) < tol
