"""The V-cycle into a caller's buffer: whatever that buffer and the solver's own hold,
0 to 2 sweeps on either side, twice in a row, against the oracle."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, fem2d, mg

from gpu_util import fixed_tensor, log, mesh_for, rel, soa, t64
from test_gpu_plane import fixed2, mesh2, soa2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [(1, 1), (2, 1), (1, 2), (2, 2), (1, 0), (0, 1)])
@pytest.mark.parametrize("plane", [False, True])
def test_vcycle_into_a_callers_buffer(nu, plane):
    log(f"vcycle dest nu={nu} plane={plane}")
    dims = (32, 16) if plane else (24, 12, 8)
    prob = synth.cantilever2d(*dims) if plane else synth.cantilever(*dims)
    kw = dict(mg_levels=3, nu_pre=nu[0], nu_post=nu[1])
    m = mesh2(prob, **kw) if plane else mesh_for(prob, **kw)
    rho = np.random.default_rng(93).uniform(0.3, 1.0, prob.n_elem)
    fixed = fixed2(prob, m) if plane else fixed_tensor(prob, m)
    m.setup(t64(rho), fixed)
    if plane:
        K, fx = fem2d.assemble2(*dims, fem.simp(rho), fem2d.q4_ke()), fem2d.fixed_dofs_aos2(prob)
    else:
        K, fx = fem.assemble(*dims, fem.simp(rho), fem.hex8_ke()), fem.fixed_dofs_aos(prob)
    H = mg.Hierarchy(K, fx, dims, 3)
    free = fem.free_mask(K.shape[0], fx)
    to_soa = soa2 if plane else soa
    r = np.random.default_rng(94).standard_normal(K.shape[0]) * free
    want = to_soa(H.vcycle(r, omega=0.6, nu1=nu[0], nu2=nu[1]))
    for _ in range(2):
        z = torch.full((K.shape[0],), float("nan"), dtype=torch.float64, device="cuda")
        m.vcycle(t64(to_soa(r)), z)
        assert rel(z.cpu().numpy(), want) < 1e-9
