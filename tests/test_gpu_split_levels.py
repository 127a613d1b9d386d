"""Split levels: supports spread so far that a level stores its flagged elements alone,
marches without them and adds them in a second launch.  Every level's product against
the fine product between interpolations; the V-cycle, with its residual and Jacobi
forms, against one that is composed of the products alone; captured ones bit by bit.
Beside them the same grids with few supports and with supports everywhere, where the
levels are not split."""

import numpy as np
import pytest
import torch

import synth

from gpu_util import log, mesh_for, t64
from test_gpu_deep_flags import _down, _up

pytestmark = pytest.mark.gpu


def _fixed(kind, dims):
    nx, ny, nz = dims
    nn = (nx + 1) * (ny + 1) * (nz + 1)
    node = torch.arange(nn, device="cuda")
    x, y, z = node % (nx + 1), node // (nx + 1) % (ny + 1), node // ((nx + 1) * (ny + 1))
    if kind == "faces":
        on = (x == 0) | (x == nx) | (y == 0) | (y == ny) | (z == 0) | (z == nz)
    else:
        share = {"spread": 0.004, "few": 0.00003, "all": 0.2}[kind]
        on = torch.rand(nn, device="cuda", generator=torch.Generator(device="cuda").manual_seed(81)) < share
    node = node[on]
    return torch.cat([c * nn + node for c in range(3)] if kind != "spread" else [(node % 3) * nn + node])


def _shape(dims, l):
    return (3, dims[2] // 2 ** l + 1, dims[1] // 2 ** l + 1, dims[0] // 2 ** l + 1)


def _composed_vcycle(m, dims, lev, mask, r, omega=0.6):
    """Algorithm 2 with one sweep each way, from the levels' products: diagonals and the
    coarsest matrix by products of unit vectors."""
    A, D = [], []
    for l in range(lev):
        n = int(np.prod(_shape(dims, l)))

        def product(v, l=l, n=n):
            y = torch.empty(n, dtype=torch.float64, device="cuda")
            m.apply(v.contiguous(), y, level=l)
            return y

        A.append(product)
        if l == lev - 1:
            K = torch.stack([product(e) for e in torch.eye(n, dtype=torch.float64, device="cuda")])
            dead = K.diagonal() == 0.0
            D.append(K + torch.diag(dead.to(torch.float64)))
            continue
        shape = _shape(dims, l)
        idx = torch.arange(n // 3, device="cuda")
        colour = (idx % shape[3]) % 3 + 3 * (idx // shape[3] % shape[2] % 3) + 9 * (idx // (shape[2] * shape[3]) % 3)
        d = torch.zeros(n, dtype=torch.float64, device="cuda")
        for c in range(3):
            for k in range(27):  # nodes of one colour share no element
                v = torch.zeros(3, n // 3, dtype=torch.float64, device="cuda")
                v[c, colour == k] = 1.0
                d += product(v.flatten()) * v.flatten()
        d[d == 0.0] = 1.0
        D.append(d)

    def cycle(l, b):
        if l == lev - 1:
            return torch.linalg.solve(D[l], b)
        x = omega * b / D[l]
        res = b - A[l](x)
        if l == 0:
            res = res * mask
        xc = cycle(l + 1, _down(res.view(_shape(dims, l))).flatten())
        e = _up(xc.view(_shape(dims, l + 1))).flatten()
        x = x + (e * mask if l == 0 else e)
        return x + omega * (b - A[l](x)) / D[l]

    return cycle(0, r)


@pytest.mark.parametrize("kind,dims,lev", [("spread", (96, 64, 96), 5), ("faces", (128, 128, 128), 6), ("spread", (16, 16, 2048), 4),
                                           ("few", (96, 64, 96), 5), ("all", (96, 64, 96), 5), ("spread", (128, 96, 128), 6)])
def test_split_levels(kind, dims, lev):
    log(f"split levels {kind} {dims} {lev}")
    prob = synth.cantilever(*dims)
    m = mesh_for(prob, mg_levels=lev)
    fixed = _fixed(kind, dims)
    rho = t64(synth.uniform_iid(*dims, 0.3, 1.0, 82).ravel())
    m.setup(rho, fixed)
    gen = torch.Generator(device="cuda").manual_seed(83)
    mask = torch.ones(m.n_dof, dtype=torch.float64, device="cuda")
    mask[fixed] = 0.0
    vs = []
    for l in range(1, lev):
        v = torch.randn(_shape(dims, l), dtype=torch.float64, device="cuda", generator=gen)
        fine = v
        for _ in range(l):
            fine = _up(fine)
        want = torch.empty(m.n_dof, dtype=torch.float64, device="cuda")
        m.apply((fine.flatten() * mask).contiguous(), want)
        want = (want * mask).view(_shape(dims, 0))
        for _ in range(l):
            want = _down(want)
        y = torch.full((v.numel(),), float("nan"), dtype=torch.float64, device="cuda")
        m.apply(v.flatten(), y, level=l)
        err = float((y - want.flatten()).norm() / want.norm())
        assert err < 1e-13 * 4 ** l, f"level {l}: {err}"  # the fine product of an interpolated vector cancels
        vs.append((v.flatten(), y))
    r = torch.randn(m.n_dof, dtype=torch.float64, device="cuda", generator=gen) * mask
    z = torch.empty_like(r)
    m.vcycle(r, z)
    want = _composed_vcycle(m, dims, lev, mask, r)
    assert float((z - want).norm() / want.norm()) < 1e-9
    # captured products choose the form on the device
    got, zc = [torch.full_like(y, float("nan")) for _, y in vs], torch.full_like(z, float("nan"))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for l, (v, _) in enumerate(vs):
            m.apply(v, got[l], level=l + 1)
        m.vcycle(r, zc)
    for _ in range(2):
        for y in got:
            y.fill_(float("nan"))
        zc.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        for l, (_, y) in enumerate(vs):
            assert torch.equal(got[l], y), f"captured level {l + 1}"
        assert torch.equal(zc, z)
    # other supports: the graph follows the next setup, split or not
    m.setup(rho, fixed[: max(3, len(fixed) // 400)])
    y = torch.empty_like(vs[0][1])
    m.apply(vs[0][0], y, level=1)
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(got[0], y)


@pytest.mark.parametrize("cases", [1, 2])
def test_fp32_cycle_on_split_levels(cases):
    """The FP32 products over the shorter lists: the first CG step as in test_gpu_fp32_cycle.py, with its bounds."""
    from paper_2205_00385_amd import aarmr

    dims, lev = (96, 64, 96), 5
    log(f"split levels fp32 x{cases}")
    prob = synth.cantilever(*dims)
    fixed = _fixed("spread", dims)
    rho = t64(synth.uniform_iid(*dims, 0.3, 1.0, 84).ravel())
    gen = torch.Generator(device="cuda").manual_seed(85)
    f, out = None, []
    for precision in (aarmr.FP64, aarmr.FP32_REFINE):
        m = mesh_for(prob, mg_levels=lev, precision=precision, cg_maxit=1, n_rhs_max=cases)
        if f is None:
            f = torch.randn(cases, m.n_dof, dtype=torch.float64, device="cuda", generator=gen)
            f[:, fixed] = 0.0
        u = torch.zeros(cases * m.n_dof, dtype=torch.float64, device="cuda")
        _, _, code = m.solve(rho, f.flatten(), fixed, u)
        assert code == aarmr.E_NOT_CONVERGED
        out.append(u.view(cases, -1))
    for l in range(cases):
        d = out[1][l] - out[0][l]
        assert float(d.norm() / out[0][l].norm()) < 3e-6
        assert float(d.abs().max() / out[0][l].abs().max()) < 3e-6
