"""A captured setup replayed with other fixed DOFs in its buffer: later eager products
and V-cycles follow the replayed setup, not the supports of the last eager one."""

import pytest
import torch

import synth

from gpu_util import log, mesh_for, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,lev", [((24, 12, 12), 3), ((48, 32, 32), 4)])
def test_eager_products_after_replays_of_a_captured_setup(dims, lev):
    log(f"captured setup {dims} {lev}")
    prob = synth.cantilever(*dims)
    m, ref = mesh_for(prob, mg_levels=lev), mesh_for(prob, mg_levels=lev)
    nn, n = m.n_node, 40
    node = torch.arange(n, device="cuda")
    few = (node % 4) * (dims[0] + 1)  # four nodes of one edge, repeated
    spread = (node * 2654435761 + 17) % nn
    gen = torch.Generator(device="cuda").manual_seed(71)
    r = torch.randn(m.n_dof, dtype=torch.float64, device="cuda", generator=gen)
    v = [torch.randn(m.dim * (dims[0] // 2 ** l + 1) * (dims[1] // 2 ** l + 1) * (dims[2] // 2 ** l + 1),
                     dtype=torch.float64, device="cuda", generator=gen) for l in range(1, lev)]
    rho = t64(synth.uniform_iid(*dims, 0.2, 1.0, 72).ravel())
    fixed = torch.cat([few, nn + few, 2 * nn + few])

    def check(nodes, replay):
        fixed.copy_(torch.cat([nodes, nn + nodes, 2 * nn + nodes]))
        if replay:
            graph.replay()
        else:
            m.setup(rho, fixed)
        ref.setup(rho, fixed)
        rz = r.clone()
        rz[fixed] = 0.0
        got, want = torch.full_like(r, float("nan")), torch.empty_like(r)
        m.vcycle(rz, got)
        ref.vcycle(rz, want)
        assert torch.equal(got, want), "V-cycle"
        for l in range(1, lev):
            y, w = torch.full_like(v[l - 1], float("nan")), torch.empty_like(v[l - 1])
            m.apply(v[l - 1], y, level=l)
            ref.apply(v[l - 1], w, level=l)
            assert torch.equal(y, w), f"level {l}"

    check(few, replay=False)  # the host has read this setup's counts
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.setup(rho, fixed)
    for nodes in (spread, few):
        check(nodes, replay=True)
    check(few, replay=False)  # an eager setup between the replays
    for nodes in (spread, few, spread):
        check(nodes, replay=True)
