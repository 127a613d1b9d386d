"""The coarsest inverse on grids whose elimination plan takes each of its
shapes: every slow axis, thin planes grouped into one block, planes of exactly
one block, of one block and a remainder, of several blocks, a single dense run,
and trees of unequal halves.  The V-cycle, whose coarsest solve is that
inverse, against the oracle's, which factors the coarsest operator directly."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, fem2d, mg

from gpu_util import aos, fixed_tensor, log, mesh_for, rel, soa, t64

pytestmark = pytest.mark.gpu

# the coarsest grid's planes (nodes along the longest axis) x unknowns per plane
CASES = [
    ((2, 2, 2), 2),     # 2 x 12: one dense run
    ((16, 2, 2), 2),    # 9 x 12, x slow: groups of five planes
    ((4, 24, 4), 2),    # 13 x 27, y slow: groups of two planes
    ((4, 8, 24), 2),    # 13 x 45, z slow
    ((6, 6, 20), 2),    # 11 x 48, z slow
    ((20, 4, 10), 2),   # 11 x 54
    ((28, 12, 4), 2),   # 15 x 63
    ((30, 8, 8), 2),    # 16 x 75: one block and a remainder
    ((24, 12, 12), 2),  # 13 x 147: three blocks a plane
    ((48, 24, 40), 4),  # 7 x 72 below three levels
]


@pytest.mark.parametrize("dims,lev", CASES)
def test_vcycle_over_elimination_plans(dims, lev):
    log(f"coarsest inverse below {dims}, {lev} levels")
    prob = synth.cantilever(*dims)
    rho = synth.uniform_iid(*dims, 0.3, 1.0, 31).ravel()
    m = mesh_for(prob, mg_levels=lev)
    m.setup(t64(rho), fixed_tensor(prob, m))
    K = fem.assemble(*dims, fem.simp(rho), fem.hex8_ke())
    fixed = fem.fixed_dofs_aos(prob)
    H = mg.Hierarchy(K, fixed, dims, lev)
    r = np.random.default_rng(32).standard_normal(K.shape[0]) * fem.free_mask(K.shape[0], fixed)
    z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
    m.vcycle(t64(soa(r)), z)
    # the coarsest operator's condition (below 1e6 for moduli in [0.027, 1])
    # times the unit roundoff, with a margin of ten
    assert rel(z.cpu().numpy(), soa(H.vcycle(r, omega=0.6, nu1=1, nu2=1))) < 1e-9


@pytest.mark.parametrize("dims", [(4, 96), (80, 40)])
def test_plane_vcycle_over_elimination_plans(dims):
    from paper_2205_00385_amd import aarmr

    log(f"coarsest inverse below {dims}, plane")
    prob = synth.cantilever2d(*dims)
    rho = np.random.default_rng(33).uniform(0.3, 1.0, prob.n_elem)
    m = aarmr.Mesh(aarmr.default_params(nx=dims[0], ny=dims[1], nz=0, mg_levels=2))
    fixed_d = torch.tensor(aarmr.fixed_dofs_soa(prob, m.n_node), dtype=torch.int64, device="cuda")
    m.setup(t64(rho), fixed_d)
    K = fem2d.assemble2(*dims, fem.simp(rho), fem2d.q4_ke())
    fixed = fem2d.fixed_dofs_aos2(prob)
    H = mg.Hierarchy(K, fixed, dims, 2)
    r = np.random.default_rng(34).standard_normal(K.shape[0]) * fem.free_mask(K.shape[0], fixed)
    z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
    m.vcycle(t64(fem2d.aos_to_soa2(r).ravel()), z)
    want = fem2d.aos_to_soa2(H.vcycle(r, omega=0.6, nu1=1, nu2=1)).ravel()
    assert rel(z.cpu().numpy(), want) < 1e-9
