"""What the autotuner tries: slabs and numberings on every lattice of the streaming
kernels (Nx = 6 to 16), the library's defaults alone on the others, and nothing that
lattice_tune refuses (runs without a GPU)."""
from types import SimpleNamespace

import pytest

from paper_1008_3647_amd import autotune


def stub(nx, ntau, dim=3):
    return SimpleNamespace(nx=nx, ntau=ntau, dim=dim)


@pytest.mark.parametrize("nx", [6, 8, 10, 12, 14, 16])
def test_streaming_lattices(nx):
    L = stub(nx, 40)
    assert autotune.candidate_slabs(L) == [1, 2, 3, 4, 6, 8]
    assert autotune.candidate_orders(L) == autotune.ORDERS
    for ntau in (2, 5, 9):
        L = stub(nx, ntau)
        assert all(1 <= s <= ntau for s in autotune.candidate_slabs(L))
        orders = autotune.candidate_orders(L)
        assert (0, False) in orders and all(g <= ntau for g, _ in orders)


@pytest.mark.parametrize("nx,ntau,dim", [(2, 40, 3), (4, 40, 3), (8, 40, 1), (16, 40, 2), (10, 40, 2),
                                         (16, 32768, 3)])
def test_other_lattices_keep_the_defaults(nx, ntau, dim):
    L = stub(nx, ntau, dim)
    assert autotune.candidate_slabs(L) == [0]
    assert autotune.candidate_orders(L) == ((-1, False),)
