"""The refinement form's FP32 V-cycle by value: the first CG step from a random load is a
multiple of the preconditioned load, so a solve stopped after one iteration returns the
V-cycle (every FP32 product of the levels, their Jacobi and residual forms, the matrices
from moments) up to FP32 rounding, where a converged solve would hide an error in it."""

import pytest
import torch

import synth

from gpu_util import fixed_tensor, log, mesh_for, t64
from test_gpu_levels import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sweeps", [(1, 1), (2, 2)])
@pytest.mark.parametrize("cases", [1, 3])
@pytest.mark.parametrize("kind,dims,lev", [
    ("face", (16, 8, 8), 3), ("corners", (24, 12, 12), 3), ("point", (24, 16, 16), 4), ("rollers", (24, 16, 16), 4),
    ("grid", (16, 12, 8), 3), ("face", (32, 16, 16), 5), ("corners", (64, 32, 32), 6),
    ("face", (128, 128, 112), 5),  # from 200,000 level-1 elements on a thread forms all 24 rows
])
def test_one_step_matches_fp64(kind, dims, lev, cases, sweeps):
    from paper_2205_00385_amd import aarmr

    log(f"fp32 cycle {kind} {dims} x{cases} sweeps={sweeps}")
    prob = _problem(kind, dims)
    rho = t64(synth.uniform_iid(*dims, 0.3, 1.0, 97).ravel())
    gen = torch.Generator(device="cuda").manual_seed(98)
    out = []
    f = None
    for precision in (aarmr.FP64, aarmr.FP32_REFINE):
        m = mesh_for(prob, mg_levels=lev, precision=precision, cg_maxit=1, n_rhs_max=cases, nu_pre=sweeps[0], nu_post=sweeps[1])
        fixed = fixed_tensor(prob, m)
        if f is None:
            f = torch.randn(cases, m.n_dof, dtype=torch.float64, device="cuda", generator=gen)
            f[:, fixed] = 0.0
        u = torch.zeros(cases * m.n_dof, dtype=torch.float64, device="cuda")
        _, st, code = m.solve(rho, f.flatten(), fixed, u)
        assert code == aarmr.E_NOT_CONVERGED and list(st.iterations)[:cases] == [1] * cases
        out.append(u.view(cases, -1))
    for l in range(cases):
        # FP32 vectors, matrices and diagonals move it by up to 3e-7 in either norm (the
        # oracle's V-cycle in FP32); one node's rows off by 10% on any level move it by 8e-6
        # in the first or 1.4e-5 in the second
        d = out[1][l] - out[0][l]
        assert float(d.norm() / out[0][l].norm()) < 3e-6
        assert float(d.abs().max() / out[0][l].abs().max()) < 3e-6
