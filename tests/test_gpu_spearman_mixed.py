"""Slices whose fluence spreads over the buckets next to one that crowds a few of them, which has all
slices ranked by sorting: the ones that stop half way leave nothing behind, wherever the crowded one is."""
import numpy as np
import pytest
import torch

from oracle import analytics as oan
from paper_2604_13929_amd import analytics as an

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,crowded", [((64, 256, 256), (0,)), ((64, 256, 256), (63,)), ((300, 100, 100), (7, 290)),
                                           ((20, 128, 120), (19,))])
def test_one_crowded_slice(shape, crowded):
    rng = np.random.default_rng(shape[0])
    f = rng.integers(0, 2 ** 45, size=shape)
    for z in crowded:                          # as few photons leave it: most voxels hold one of three values
        f[z] = np.where(rng.random(shape[1:]) < 0.02, f[z], 2 ** 31 * rng.integers(1, 4, size=shape[1:]))
        f[z, 0, 0] = 0
    m = (rng.random(shape) < 0.7).astype(np.uint8)
    rho, n = an.pore_spearman(torch.from_numpy(m).cuda(), torch.from_numpy(f).cuda(), 0)
    want, nw = oan.pore_spearman(f, m, 0)
    assert np.array_equal(n.cpu().numpy(), nw)
    assert np.all(np.abs(rho.cpu().numpy() - want) <= 1e-12)
