"""The filter and its adjoint in LDS tiles of 32 x 8 elements by one, two or four
layers: one element less and more than a tile on each axis, single layers, grids
thinner than the reach, and the reach where the per-element kernel takes over."""

import numpy as np
import pytest
import torch

from oracle import filt

from gpu_util import log, rel, t64
from paper_2205_00385_amd import aarmr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2), (32, 8, 4), (34, 10, 6), (30, 6, 2), (64, 16, 8), (66, 18, 10), (32, 8, 0), (34, 18, 0)])
@pytest.mark.parametrize("r", [1.5, 2.0, 2.5, 3.0, 3.5])
def test_filter_tiles_match_oracle(dims, r):
    log(f"filter tiles {dims} r={r}")
    m = aarmr.Mesh(aarmr.default_params(nx=dims[0], ny=dims[1], nz=dims[2], mg_levels=2, rmin=r))
    H, Hs = filt.filter_matrix(dims[0], dims[1], max(dims[2], 1), r)
    x = np.random.default_rng(91).uniform(-1.0, 1.0, m.n_elem)
    y = torch.full((m.n_elem,), float("nan"), dtype=torch.float64, device="cuda")
    m.filter(t64(x), y, mode=0)
    assert rel(y.cpu().numpy(), filt.forward(H, Hs, x)) < 1e-13  # sums of at most 125 terms
    m.filter(t64(x), y, mode=1)
    assert rel(y.cpu().numpy(), filt.adjoint(H, Hs, x)) < 1e-13
