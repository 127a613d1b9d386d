"""The OC bisection in launches of five steps: grids around one workgroup's elements,
a damping exponent other than 1/2, a first call whose guess of the launch count is too
small (a tiny multiplier takes more steps), x updated in place, and volumes on which
every step turns the same way, against the oracle."""

import numpy as np
import pytest
import torch

import synth
from oracle import filt, oc

from gpu_util import log, mesh_for, rel, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,eta,scale,volfrac", [
    ((4, 2, 2), 0.5, 1.0, 0.4),
    ((8, 8, 8), 0.5, 1.0, 0.3),        # 512 elements: one workgroup's threads
    ((36, 12, 8), 0.3, 1.0, 0.35),
    ((64, 48, 44), 0.5, 1.0, 0.3),     # 135,168 elements: more than one per thread
    ((8, 6, 4), 0.5, 1e-9, 0.3),       # sensitivities of 1e-9: about 30 steps more
    ((8, 6, 4), 0.5, 1e-40, 0.3),
    ((8, 6, 4), 0.5, 1.0, 0.999),      # out of reach: the multiplier falls until the 200th step
    ((8, 6, 4), 0.5, 1.0, 0.001),      # out of reach: it rises to the upper end
])
def test_oc_rounds_match_oracle(dims, eta, scale, volfrac):
    log(f"oc rounds {dims} eta={eta} scale={scale} volfrac={volfrac}")
    m = mesh_for(synth.cantilever(*dims), mg_levels=2 if dims[0] < 36 else 3, rmin=2.0, oc_eta=eta)
    H, Hs = filt.filter_matrix(*dims, 2.0)
    rng = np.random.default_rng(81)
    x = rng.uniform(0.1, 0.9, m.n_elem)
    dc = -scale * rng.uniform(0.01, 3.0, m.n_elem)
    dv = filt.adjoint(H, Hs, np.ones(m.n_elem))
    xn, xp, _ = oc.oc_update(x, dc, dv, H, Hs, volfrac, eta=eta)
    gx = torch.full((m.n_elem,), float("nan"), dtype=torch.float64, device="cuda")
    gp = torch.full_like(gx, float("nan"))
    for _ in range(2):  # the second call knows the number of launches
        m.oc_update(t64(x), t64(dc), t64(dv), volfrac, 0.2, gx, gp)
        assert rel(gx.cpu().numpy(), xn) < 1e-9
        assert rel(gp.cpu().numpy(), xp) < 1e-9
    fresh = mesh_for(synth.cantilever(*dims), mg_levels=2 if dims[0] < 36 else 3, rmin=2.0, oc_eta=eta)
    d = t64(x)
    s = t64(dc)
    fresh.oc_update(d, s, t64(dv), volfrac, 0.2, d, s)  # outputs over the inputs
    assert torch.equal(d, gx) and torch.equal(s, gp)
    m.oc_update_noalloc(t64(x), t64(dc), t64(dv), volfrac, 0.2, d, s)
    assert torch.equal(d, gx) and torch.equal(s, gp)
