"""Hierarchies of six to eight levels, whose deep elements stand for rows of 16 to 64
level-1 flags: every level's product against the fine product between interpolations,
with single fixed DOFs that a deep element meets at its first, last or middle row."""

import pytest
import torch

import synth

from gpu_util import log, mesh_for, t64

pytestmark = pytest.mark.gpu


def _up(v):  # trilinear interpolation to the 2:1 refined grid, [3][z][y][x]
    for axis in (1, 2, 3):
        n = v.shape[axis]
        shape = list(v.shape)
        shape[axis] = 2 * n - 1
        out = torch.empty(shape, dtype=v.dtype, device=v.device)
        lo, hi = v.narrow(axis, 0, n - 1), v.narrow(axis, 1, n - 1)
        idx = torch.arange(n, device=v.device)
        out.index_copy_(axis, 2 * idx, v)
        out.index_copy_(axis, 2 * idx[:-1] + 1, 0.5 * (lo + hi))
        v = out
    return v


def _down(v):  # its transpose
    for axis in (1, 2, 3):
        n = (v.shape[axis] + 1) // 2
        idx = torch.arange(n, device=v.device)
        out = v.index_select(axis, 2 * idx)
        odd = 0.5 * v.index_select(axis, 2 * idx[:-1] + 1)
        out.narrow(axis, 0, n - 1).add_(odd)
        out.narrow(axis, 1, n - 1).add_(odd)
        v = out
    return v


@pytest.mark.parametrize("dims,lev", [((64, 32, 32), 6), ((128, 64, 64), 7), ((128, 128, 128), 8)])
@pytest.mark.parametrize("kind", ["last", "first", "middle"])
def test_levels_match_the_interpolated_fine_product(dims, lev, kind):
    log(f"deep flags {dims} {lev} {kind}")
    nx, ny, nz = dims
    m = mesh_for(synth.cantilever(*dims), mg_levels=lev)
    at = {"last": (nx, ny, nz), "first": (0, 0, 0), "middle": (nx // 2 - 1, ny // 4 + 1, 3 * nz // 4 - 3)}[kind]
    node = at[0] + (nx + 1) * (at[1] + (ny + 1) * at[2])
    fixed = torch.tensor([c * m.n_node + node for c in range(3)] + [m.n_node + node - 1 if node else 1], device="cuda")
    rho = t64(synth.uniform_iid(*dims, 0.3, 1.0, 61).ravel())
    m.setup(rho, fixed)
    gen = torch.Generator(device="cuda").manual_seed(62)
    for l in range(1, lev):
        shape = (3, nz // 2 ** l + 1, ny // 2 ** l + 1, nx // 2 ** l + 1)
        v = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
        fine = v
        for _ in range(l):
            fine = _up(fine)
        fine = fine.flatten()
        fine[fixed] = 0.0
        want = torch.empty_like(fine)
        m.apply(fine, want)
        want[fixed] = 0.0
        want = want.view(3, nz + 1, ny + 1, nx + 1)
        for _ in range(l):
            want = _down(want)
        y = torch.full((v.numel(),), float("nan"), dtype=torch.float64, device="cuda")
        m.apply(v.flatten(), y, level=l)
        # the fine product of an interpolated vector cancels by a factor of about 4^l
        err = float((y - want.flatten()).norm() / want.norm())
        assert err < 1e-13 * 4 ** l, f"level {l}: {err}"
