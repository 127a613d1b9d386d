"""Default launch shapes of the fine-grid product, from a grid thinner than one chunk
to one whose tiles fill the device: each against one chunk of 16-row tiles, whose bits
it has to repeat, and the small ones against the oracle's assembled matrix."""

import numpy as np
import pytest
import torch

import synth
from oracle import fem

from gpu_util import aos, fixed_tensor, log, mesh_for, rel, soa, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2), (4, 14, 2), (30, 8, 6), (28, 6, 16), (32, 16, 10), (60, 28, 36), (96, 48, 48),
                                  (104, 56, 40), (128, 64, 64)])
@pytest.mark.parametrize("masked", [False, True])
def test_default_shape_repeats_the_bits_of_one_chunk(dims, masked):
    from paper_2205_00385_amd import aarmr

    log(f"shapes {dims} masked={masked}")
    prob = synth.cantilever(*dims)
    rho = synth.uniform_iid(*dims, 0.1, 1.0, 71).ravel()
    m = mesh_for(prob, mg_levels=2 if dims[0] < 60 else 3 if dims[0] < 96 else 4)
    fixed = fixed_tensor(prob, m)
    m.setup(t64(rho), fixed)
    v = torch.randn(m.n_dof, dtype=torch.float64, generator=torch.Generator().manual_seed(72)).cuda()
    if masked:
        v[fixed] = 0.0
    flags = aarmr.INPUT_MASKED if masked else 0
    y, one = torch.full_like(v, float("nan")), torch.full_like(v, float("nan"))
    m.apply(v, y, flags=flags)
    m.set_chunk((16 << 16) | (dims[2] + 1))
    m.apply(v, one, flags=flags)
    assert torch.equal(y, one)
    if m.n_dof < 20000:
        free = fem.free_mask(m.n_dof, fem.fixed_dofs_aos(prob))
        a = aos(v.cpu().numpy())
        want = (fem.assemble(*dims, fem.simp(rho), fem.hex8_ke()) @ (a * free)) * free
        if not masked:
            want = want + a * (1 - free)
        assert rel(y.cpu().numpy(), soa(want)) < 1e-13  # sums of 192 products in another order
