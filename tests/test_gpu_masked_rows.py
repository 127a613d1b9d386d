"""The FP32 level-1 product's flagged parents in twelve-row workgroups: supports from
one DOF (a list of a few entries, an odd workgroup left over) to a support in every
level-1 element, through refinement-form solves against the FP64 form."""

import pytest
import torch

import synth

from gpu_util import fixed_tensor, loads_tensor, log, mesh_for, rel, t64
from test_gpu_levels import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,dims,lev", [("face", (16, 8, 8), 3), ("corners", (24, 12, 12), 3), ("point", (24, 16, 16), 4),
                                           ("rollers", (24, 16, 16), 4), ("grid", (16, 12, 8), 3)])
def test_refinement_form_matches_fp64_for_all_supports(kind, dims, lev):
    from paper_2205_00385_amd import aarmr

    log(f"masked rows {kind} {dims}")
    prob = _problem(kind, dims)
    rho = t64(synth.uniform_iid(*dims, 0.3, 1.0, 97).ravel())
    out = []
    for precision in (aarmr.FP64, aarmr.FP32_REFINE):
        m = mesh_for(prob, mg_levels=lev, precision=precision, cg_rtol=1e-9)
        f = loads_tensor(prob, m)
        u = torch.zeros_like(f)
        _, _, code = m.solve(rho, f, fixed_tensor(prob, m), u)
        assert code == 0
        out.append(u.cpu().numpy())
    # residuals of 1e-9 times condition numbers of up to about 1e3 on these supports' solutions
    assert rel(out[1], out[0]) < 1e-6
