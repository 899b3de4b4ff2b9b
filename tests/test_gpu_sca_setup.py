"""The strong-coupling factors where the chunked setup is delicate: alpha = 1 (one
row of a chunk's matrix stays constant while the other is a product of all b_t^2),
long time extents at strong coupling and constant fields (that product leaves the
exponent range), fields whose b^2 stays above 1 and then below it (E_t = D_t -
b_t^2 decays below the rounding of D and grows back), alpha below 1, and
magnitudes beyond what a chunk rescales.

Reference: the recursions of the oracle and the two sweeps in long double.
Tolerance: that of every strong-coupling application (complex128 1e-12, complex64
2e-5), or, where the smallest D makes the recursion itself less accurate, 16
roundings of the largest D against the smallest, or 16 times the error of the same
recursions in double precision.
"""
import numpy as np
import pytest
import torch

from oracle import precond as pc
from oracle.operator import coupling_A
from gpu_util import require_gpu, to_dev, to_host, rel_err, say, TAU

pytestmark = pytest.mark.gpu

NX = 2


def field(kind, ntau):
    rng = np.random.default_rng(611)
    if kind == "iid":
        return rng.uniform(-np.pi, np.pi, size=(ntau, NX))
    if kind == "constant":
        return np.full((ntau, NX), np.pi / 2)
    s = rng.uniform(0.9, 1.0, size=(ntau, NX))  # b = 1.7 and more, then 0.3 and less
    s[ntau // 2:] *= -0.9
    return np.arcsin(s)


def reference(sigma, g, alpha, v, real):
    """x by the recursions in the precision of `real`, and the factors D."""
    b = (1.0 + coupling_A(TAU, g) * np.sin(sigma)).astype(real)
    D, L = pc.sca_factor(b, real(alpha))
    w = v.astype(np.clongdouble if real is np.longdouble else np.complex128)
    for t in range(1, len(b)):
        w[t] = v[t] + L[t - 1] * w[t - 1]
    w[-1] -= L[-1] * v[0]
    w = w / D
    for t in range(len(b) - 2, -1, -1):
        w[t] = w[t] + L[t] * w[t + 1]
    w[0] -= L[-1] * w[-1]
    return w, D


def applied(sigma, g, alpha, v, dtype):
    from paper_1008_3647_amd import Lattice, Precond
    L = Lattice(NX, len(sigma), TAU, g, dtype, dim=1)
    L.set_aux_field(to_dev(sigma))
    return to_host(L.apply_precond(to_dev(v[None], dtype), Precond("sca", alpha=alpha), "Q"))[0]


def vector(ntau):
    rng = np.random.default_rng(612)
    v = rng.standard_normal((ntau, NX)) + 1j * rng.standard_normal((ntau, NX))
    return v.astype(np.complex64).astype(np.complex128)


@pytest.mark.parametrize("kind,g,ntau,alpha,dtypes", [
    ("iid", 5.0, 40, 1.0, "sd"), ("iid", 5.0, 1000, 1.0, "sd"),
    ("iid", 80.0, 8000, 1.0, "sd"), ("iid", 80.0, 16000, 1.0, "sd"),
    ("constant", 40.0, 8000, 1.0, "sd"), ("constant", 5.0, 24000, 1.0, "sd"),
    ("iid", 80.0, 8000, 1.0 + 1e-12, "d"), ("iid", 80.0, 8000, 3.0, "sd"),
    ("iid", 5.0, 200, 0.5, "d"), ("iid", 5.0, 1000, 0.05, "d"), ("iid", 80.0, 300, 0.9, "d"),
    ("iid", 5.0, 300, 1e12, "d"), ("iid", 5.0, 300, 1e40, "d"), ("iid", 1600.0, 300, 1.0, "d"),
])
def test_sca_factors(kind, g, ntau, alpha, dtypes):
    require_gpu()
    sigma, v = field(kind, ntau), vector(ntau)
    ref, D = reference(sigma, g, alpha, v, np.longdouble)
    double = rel_err(reference(sigma, g, alpha, v, np.float64)[0], ref)
    rounding = float(2.0 ** -53 * np.max(np.abs(D)) / np.min(np.abs(D)))
    for dtype, tol in ((torch.complex64, 2e-5), (torch.complex128, 1e-12)):
        if ("s" if dtype == torch.complex64 else "d") not in dtypes:
            continue
        tol = max(tol, 16 * rounding, 16 * double)
        say(f"sca factors {kind} g={g} ntau={ntau} alpha={alpha} {dtype} tol={tol:.1e}")
        y = applied(sigma, g, alpha, v, dtype)
        assert np.isfinite(y).all()
        err = rel_err(y, ref)
        say(f"  {err:.1e}")
        assert err < tol


def test_sca_factors_regrowing():
    """E decays by 4^-400 and grows back: what the recursion returns is its rounding,
    so only the size is compared; exact E would give vectors of 1e91."""
    require_gpu()
    ntau, g = 800, 5.0
    sigma, v = field("regrowing", ntau), vector(ntau)
    size = np.max(np.abs(reference(sigma, g, 1.0, v, np.float64)[0]))
    for dtype in (torch.complex64, torch.complex128):
        say(f"sca factors regrowing {dtype}")
        y = applied(sigma, g, 1.0, v, dtype)
        say(f"  {np.max(np.abs(y)):.1e} (double recursion {size:.1e})")
        assert np.isfinite(y).all()
        assert 1e-3 * size < np.max(np.abs(y)) < 1e3 * size
