"""Graph capture of the V-cycle and of the products on every level, right after a setup
and with no call in between: replays give the eager call's bits, also after another
setup with other fixed DOFs, with the program's own work between the replays."""

import numpy as np
import pytest
import torch

import synth

from gpu_util import fixed_tensor, log, mesh_for, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,lev", [((24, 12, 12), 3), ((48, 32, 32), 4)])
def test_captured_vcycle_follows_the_setup(dims, lev):
    log(f"capture {dims} {lev}")
    prob = synth.cantilever(*dims)
    m, eager = mesh_for(prob, mg_levels=lev), mesh_for(prob, mg_levels=lev)
    face = fixed_tensor(prob, m)
    node = m.n_node // 2 + 3
    more = torch.cat([face, torch.tensor([node, m.n_node + 7, 2 * m.n_node + node + 5], device="cuda")])
    rng = np.random.default_rng(95)
    r = t64(rng.standard_normal(m.n_dof))
    z = torch.zeros_like(r)
    v = [t64(rng.standard_normal(3 * int(np.prod([d // 2 ** l + 1 for d in dims])))) for l in range(1, lev)]
    y = [torch.zeros_like(a) for a in v]
    for k, fixed in enumerate((face, more, face[: len(face) // 2])):
        rho = t64(rng.uniform(0.2, 1.0, m.n_elem))
        for mesh in (m, eager):
            mesh.setup(rho, fixed)
        torch.cuda.synchronize()
        if k == 0:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                m.vcycle(r, z)
                for l in range(1, lev):
                    m.apply(v[l - 1], y[l - 1], level=l)
        for _ in range(2):
            z.fill_(float("nan"))
            r.copy_(t64(rng.standard_normal(m.n_dof)))
            r[fixed] = 0.0
            g.replay()
            torch.cuda.synchronize()
            want = torch.empty_like(z)
            eager.vcycle(r, want)
            assert torch.equal(z, want)
            for l in range(1, lev):
                wl = torch.empty_like(y[l - 1])
                eager.apply(v[l - 1], wl, level=l)
                assert torch.equal(y[l - 1], wl), f"level {l}"
