"""Coarse-level operators in moment form, with the stored matrices around fixed
DOFs: every level's product, and the V-cycle that uses its residual and Jacobi
forms, against the oracle's assembled hierarchy.  The supports cover what the
lists have to tell apart: a whole face, rollers on three faces (single components
fixed), four corner nodes, one component of one interior node, and every node of a
level special."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, mg

from gpu_util import aos, fixed_tensor, log, mesh_for, rel, soa, t64

pytestmark = pytest.mark.gpu


def _problem(kind, dims):
    nx, ny, nz = dims
    if kind == "face":
        return synth.cantilever(*dims)
    if kind == "rollers":
        return synth.patch_test(*dims)
    if kind == "corners":
        return synth.bridge(*dims)
    prob = synth.cantilever(*dims)
    if kind == "point":  # a support inside the grid, in y only, beside a clamped corner
        prob.fixed = [(nx // 2 + 1, ny // 2, nz // 2, 1)] + [(0, 0, 0, c) for c in range(3)] + [(nx, 0, 0, 2), (0, ny, 0, 0), (0, 0, nz, 1)]
    else:  # "grid": a support in every element of the level below the finest
        prob.fixed = [(i, j, k, (i + j + k) % 3) for i in range(1, nx, 2) for j in range(1, ny, 2) for k in range(1, nz, 2)]
    return prob


@pytest.mark.parametrize("kind,dims,lev", [
    ("face", (8, 4, 4), 3),
    ("face", (72, 12, 20), 3),      # 36 x 6 x 10: two tiles along x, a partial one along y
    ("rollers", (24, 16, 16), 4),
    ("corners", (24, 36, 12), 3),   # 12 x 18 x 6: three tiles along y
    ("point", (40, 24, 32), 4),
    ("grid", (16, 12, 8), 3),
])
@pytest.mark.parametrize("field", ["iid", "contrast"])
def test_levels_match_oracle(kind, dims, lev, field):
    log(f"levels {kind} {dims} {lev} {field}")
    prob = _problem(kind, dims)
    if field == "iid":
        rho = synth.uniform_iid(*dims, 0.3, 1.0, 51).ravel()
    else:  # moduli 1e-9 and 1 side by side
        rho = synth.thresholded_field(*dims, 1.5, 1e-3, 1.0, 52).ravel()
    m = mesh_for(prob, mg_levels=lev)
    m.setup(t64(rho), fixed_tensor(prob, m))
    K = fem.assemble(*dims, fem.simp(rho), fem.hex8_ke())
    fixed = fem.fixed_dofs_aos(prob)
    H = mg.Hierarchy(K, fixed, dims, lev)
    rng = np.random.default_rng(53)
    for l in range(1, lev):
        nn = int(np.prod([d // 2 ** l + 1 for d in dims]))
        v = rng.standard_normal(3 * nn)
        y = torch.full((3 * nn,), float("nan"), dtype=torch.float64, device="cuda")
        m.apply(t64(v), y, level=l)
        # sums of a few hundred products in another order: 1e-12 with a wide margin
        assert rel(y.cpu().numpy(), soa(H.A[l] @ aos(v))) < 1e-12, f"level {l}"
    if field == "iid":
        r = rng.standard_normal(K.shape[0]) * fem.free_mask(K.shape[0], fixed)
        z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
        m.vcycle(t64(soa(r)), z)
        want = soa(H.vcycle(r, omega=0.6, nu1=1, nu2=1))
        assert rel(z.cpu().numpy(), want) < 1e-9
