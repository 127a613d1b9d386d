"""Levels of up to 11 elements along x, whose products run a tile per wavefront: grids
with one and two tiles along x and along y, the last one partial, and numbers of chunks
that leave wavefronts of the last workgroup without one.  Every level's product, and
the V-cycle with its residual and Jacobi forms, against the oracle's hierarchy."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, mg

from gpu_util import aos, fixed_tensor, log, mesh_for, rel, soa, t64
from test_gpu_levels import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,dims,lev", [
    ("face", (8, 8, 64), 3),      # level 1 4 x 4 x 32: one tile
    ("corners", (12, 28, 40), 3), # 6 x 14 x 20: two tiles along x, three along y
    ("point", (20, 12, 36), 3),   # 10 x 6 x 18: a partial tile along x, exactly one along y
    ("rollers", (16, 16, 160), 4),  # 8 x 8 x 80 and, from moments, 4 x 4 x 40
    ("grid", (16, 32, 16), 4),
    ("face", (32, 16, 64), 4),    # a wide level above a narrow one
])
@pytest.mark.parametrize("sweeps", [(1, 1), (2, 2)])
def test_narrow_levels_match_oracle(kind, dims, lev, sweeps):
    log(f"narrow levels {kind} {dims} {lev} {sweeps}")
    prob = _problem(kind, dims)
    rho = synth.uniform_iid(*dims, 0.3, 1.0, 41).ravel()
    m = mesh_for(prob, mg_levels=lev, nu_pre=sweeps[0], nu_post=sweeps[1])
    m.setup(t64(rho), fixed_tensor(prob, m))
    K = fem.assemble(*dims, fem.simp(rho), fem.hex8_ke())
    fixed = fem.fixed_dofs_aos(prob)
    H = mg.Hierarchy(K, fixed, dims, lev)
    rng = np.random.default_rng(42)
    for l in range(1, lev):
        nn = int(np.prod([d // 2 ** l + 1 for d in dims]))
        v = rng.standard_normal(3 * nn)
        y = torch.full((3 * nn,), float("nan"), dtype=torch.float64, device="cuda")
        m.apply(t64(v), y, level=l)
        assert rel(y.cpu().numpy(), soa(H.A[l] @ aos(v))) < 1e-12, f"level {l}"
    r = rng.standard_normal(K.shape[0]) * fem.free_mask(K.shape[0], fixed)
    z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
    m.vcycle(t64(soa(r)), z)
    assert rel(z.cpu().numpy(), soa(H.vcycle(r, omega=0.6, nu1=sweeps[0], nu2=sweeps[1]))) < 1e-9
