"""autotune on a lattice that streams without being a multiple of 4 (Nx = 10): every
slab and numbering is timed, a choice stored for earlier kernels is not taken, and a
tuned lattice gives the untuned one's weak-coupling application bit for bit."""
import json

import pytest
import torch

from synthetic import sigma_field, gaussian_rhs
from gpu_util import require_gpu, to_dev, say, TAU, G

pytestmark = pytest.mark.gpu


def test_tune_nx10(tmp_path):
    require_gpu()
    from paper_1008_3647_amd import Lattice, Precond
    from paper_1008_3647_amd import autotune as at
    nx, ntau = 10, 12
    L = Lattice(nx, ntau, TAU, G, torch.complex128)
    L.set_aux_field(to_dev(sigma_field(nx, ntau, 701)))
    b = to_dev(gaussian_rhs(nx, ntau, [702, 703]))
    p = Precond("wce", wce_order=2)
    ref = L.apply_precond(b, p, "M")
    cache = tmp_path / "tune.json"
    key = at._key(L, 2, False, p)
    old = dict(slab=7, vec_blocks=3, xcd_group=0, rhs_inner=False, seconds=1.0)
    cache.write_text(json.dumps({"v3|" + key: old}))
    kw = dict(iters=4, reps=1, vec_blocks=(0, 64), refine_reps=0, precond=p, cache=str(cache))
    t = at.tune(L, b, **kw)
    say({k: t[k] for k in ("slab", "vec_blocks", "xcd_group", "rhs_inner")})
    assert not t["cached"]
    assert len(t["candidates"]) == len(at.candidate_slabs(L)) * len(at.ORDERS) + 1
    assert torch.equal(L.apply_precond(b, p, "M"), ref)
    again = at.tune(L, b, **kw)
    assert again["cached"] and all(again[k] == t[k] for k in ("slab", "vec_blocks", "xcd_group"))
    t = at.tune_apply(L, b, launches=3, reps=1)
    assert len(t["candidates"]) == len(at.candidate_slabs(L)) * len(at.ORDERS)
    assert torch.equal(L.apply_precond(b, p, "M"), ref)
