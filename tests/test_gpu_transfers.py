"""Transfers of the V-cycle at both sides of the interpolation's split into single
components (256 workgroups of 256 fine nodes; 60x36x28 has 65,453 nodes, just
enough): masks, partial workgroups and the coarsest order, against the oracle."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, mg

from gpu_util import aos, fixed_tensor, log, mesh_for, rel, soa, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,lev", [((60, 36, 28), 3), ((60, 36, 24), 3), ((4, 2, 2), 2)])
def test_vcycle_around_the_component_split(dims, lev):
    log(f"transfers {dims} {lev}")
    prob = synth.cantilever(*dims)
    rho = synth.uniform_iid(*dims, 0.3, 1.0, 61).ravel()
    m = mesh_for(prob, mg_levels=lev)
    m.setup(t64(rho), fixed_tensor(prob, m))
    K = fem.assemble(*dims, fem.simp(rho), fem.hex8_ke())
    fixed = fem.fixed_dofs_aos(prob)
    H = mg.Hierarchy(K, fixed, dims, lev)
    r = np.random.default_rng(62).standard_normal(K.shape[0]) * fem.free_mask(K.shape[0], fixed)
    z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
    m.vcycle(t64(soa(r)), z)
    want = soa(H.vcycle(r, omega=0.6, nu1=1, nu2=1))
    assert rel(z.cpu().numpy(), want) < 1e-9
