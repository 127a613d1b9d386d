"""Plane-stress products where a workgroup takes several groups of 64 nodes (above
65,536 nodes) and where the last group is partial: the fine operator in both input
forms, every level and the V-cycle against the oracle, and the solver's own sweep and
dot products through a solve whose residual is formed by the oracle's matrix."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem, mg

from gpu_util import log, rel, t64
from test_gpu_plane import aos2, density2, fixed2, loads2, mesh2, operator2, soa2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,lev", [(62, 2, 2), (256, 248, 4), (256, 256, 5), (512, 256, 6)])
def test_plane_products_over_node_groups(nx, ny, lev):
    from paper_2205_00385_amd import aarmr

    log(f"plane products {nx}x{ny} levels={lev}")
    prob = synth.cantilever2d(nx, ny)
    rho = density2(prob, 31)
    m = mesh2(prob, mg_levels=lev, cg_rtol=1e-8)
    m.setup(t64(rho), fixed2(prob, m))
    K, fixed, A = operator2(prob, rho)
    rng = np.random.default_rng(32)
    v = rng.standard_normal(2 * m.n_node)
    y = torch.full((2 * m.n_node,), float("nan"), dtype=torch.float64, device="cuda")
    m.apply(t64(v), y)
    assert rel(y.cpu().numpy(), soa2(A @ aos2(v))) < 1e-13
    free = fem.free_mask(K.shape[0], fixed)
    vm = aos2(v) * free
    m.apply(t64(soa2(vm)), y, flags=aarmr.INPUT_MASKED)
    assert rel(y.cpu().numpy(), soa2(A @ vm)) < 1e-13
    H = mg.Hierarchy(K, fixed, (nx, ny), lev)
    for l in range(1, lev):
        nn = (nx // 2 ** l + 1) * (ny // 2 ** l + 1)
        w = rng.standard_normal(2 * nn)
        yl = torch.full((2 * nn,), float("nan"), dtype=torch.float64, device="cuda")
        m.apply(t64(w), yl, level=l)
        assert rel(yl.cpu().numpy(), soa2(H.A[l] @ aos2(w))) < 1e-12, f"level {l}"
    r = rng.standard_normal(K.shape[0]) * free
    z = torch.zeros(K.shape[0], dtype=torch.float64, device="cuda")
    m.vcycle(t64(soa2(r)), z)
    assert rel(z.cpu().numpy(), soa2(H.vcycle(r, omega=0.6, nu1=1, nu2=1))) < 1e-9
    f = loads2(prob, m)
    u = torch.zeros_like(f)
    _, _, code = m.solve(t64(rho), f, fixed2(prob, m), u)
    assert code == 0
    fa = aos2(f.cpu().numpy()) * free
    assert np.linalg.norm(fa - A @ aos2(u.cpu().numpy())) <= 2e-8 * np.linalg.norm(fa)
