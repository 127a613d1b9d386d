"""Reduced models whose K_Phi products don't fit one reduction (Ns > Nm + 1) and whose
Gram-Schmidt runs over several columns, on both grids, against the oracle's eqs. 15-29."""

import numpy as np
import pytest
import torch

import synth
from oracle import ca as oca
from oracle import fem, fem2d, solve

from gpu_util import fixed_tensor, loads_tensor, log, mesh_for, rel, soa, t64
from test_gpu_plane import fixed2, loads2, mesh2, operator2, soa2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ns,Nm", [(2, 1), (1, 2), (4, 2), (3, 3)])
@pytest.mark.parametrize("plane", [False, True])
def test_ca_update_over_basis_sizes(Ns, Nm, plane):
    from paper_2205_00385_amd import aarmr

    log(f"ca groups Ns={Ns} Nm={Nm} plane={plane}")
    kw = dict(mg_levels=3, cg_rtol=1e-11, Ns=Ns, Nm=Nm, ca_tol=1.0)
    prob = synth.cantilever2d(48, 24) if plane else synth.cantilever(16, 8, 8)
    m = mesh2(prob, **kw) if plane else mesh_for(prob, **kw)
    fixed_t = fixed2(prob, m) if plane else fixed_tensor(prob, m)
    f = loads2(prob, m) if plane else loads_tensor(prob, m)
    rng = np.random.default_rng(98)
    base, drift = rng.uniform(0.4, 1.0, prob.n_elem), rng.uniform(-1.0, 1.0, (Ns + 1, prob.n_elem))
    designs = [np.clip(base + 0.02 * d, 0.05, 1.0) for d in drift]

    def system(rho):
        if plane:
            K, fx, A = operator2(prob, rho)
        else:
            K = fem.assemble(prob.nx, prob.ny, prob.nz, fem.simp(rho), fem.hex8_ke())
            fx = fem.fixed_dofs_aos(prob)
            A = fem.operator_with_bc(K, fx)
        load = (fem2d.dof_vector_aos2(prob) if plane else fem.dof_vector_aos(prob, 0)) * fem.free_mask(A.shape[0], fx)
        if plane:
            return A, load, fem2d.analyse2(prob, rho)[0][0]
        return A, load, solve.solve_direct(K, load, fx, (prob.nx, prob.ny, prob.nz))

    u = torch.zeros_like(f)
    Phi = []
    for k in range(Ns):
        A_prev, _, u_last = system(designs[k])
        Phi = oca.parm_fifo(Phi, u_last, Ns)
        m.solve(t64(designs[k]), f, fixed_t, u, flags=aarmr.RECORD_PARM | (aarmr.WARM_START if k else 0))
    A, load, _ = system(designs[Ns])
    want, eps, rank = oca.ca_approximation(A, A_prev, np.stack(Phi, axis=1), u_last, load, Nm)
    _, st, _ = m.ca_update(t64(designs[Ns]), f, fixed_t, u)
    log(f"  eps gpu={st.eps[0]:.6e} oracle={eps:.6e} rank {st.rank[0]}/{rank}")
    assert st.rank[0] == rank
    assert abs(st.eps[0] - eps) <= 1e-6 * eps + 1e-12
    assert rel(u.cpu().numpy(), (soa2 if plane else soa)(want)) < 1e-6
