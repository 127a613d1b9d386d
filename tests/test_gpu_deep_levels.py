"""Hierarchies of five and six levels, where moments are shifted from level to level,
and moduli 1e-9 and 1 side by side, where they cancel most: every row of every level's
product, and the V-cycle with the Jacobi diagonals, against the oracle's hierarchy."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, mg

from gpu_util import aos, fixed_tensor, log, mesh_for, rel, soa, t64
from test_gpu_levels import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,dims,lev", [("face", (32, 16, 16), 5), ("rollers", (32, 16, 16), 5), ("point", (32, 32, 48), 5),
                                           ("corners", (64, 32, 32), 6), ("grid", (16, 32, 16), 5)])
@pytest.mark.parametrize("field", ["iid", "contrast"])
def test_rows_of_deep_levels_match_oracle(kind, dims, lev, field):
    log(f"deep levels {kind} {dims} {lev} {field}")
    prob = _problem(kind, dims)
    if field == "iid":
        rho = synth.uniform_iid(*dims, 0.3, 1.0, 51).ravel()
    else:
        rho = synth.thresholded_field(*dims, 1.5, 1e-3, 1.0, 52).ravel()
    m = mesh_for(prob, mg_levels=lev)
    m.setup(t64(rho), fixed_tensor(prob, m))
    K = fem.assemble(*dims, fem.simp(rho), fem.hex8_ke())
    fixed = fem.fixed_dofs_aos(prob)
    H = mg.Hierarchy(K, fixed, dims, lev)
    rng = np.random.default_rng(53)
    for l in range(1, lev):
        nn = int(np.prod([d // 2 ** l + 1 for d in dims]))
        v = rng.uniform(-1.0, 1.0, 3 * nn)
        y = torch.full((3 * nn,), float("nan"), dtype=torch.float64, device="cuda")
        m.apply(t64(v), y, level=l)
        # a moment carries its whole element: against the diagonal of a corner that sees
        # only the far side of one stiff descendant, its rounding is larger by (2^l)^4
        err = np.abs(aos(y.cpu().numpy()) - H.A[l] @ aos(v)) / H.D[l]
        live = H.A[l] @ np.ones(3 * nn) != 1.0  # identity rows of dead coarse DOFs aside
        assert err[live].max() < 64 * 1.1e-16 * 16 ** l, f"level {l}: {err[live].max()}"
    r = rng.standard_normal(K.shape[0]) * fem.free_mask(K.shape[0], fixed)
    z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
    m.vcycle(t64(soa(r)), z)
    got, want = aos(z.cpu().numpy()), H.vcycle(r, omega=0.6, nu1=1, nu2=1)
    # entries off by that rounding move it by 3e-13 in this norm; one diagonal off by 10%
    # moves it by 5e-9 or more
    w = np.sqrt(H.D[0])
    assert rel(w * got, w * want) < 1e-10
