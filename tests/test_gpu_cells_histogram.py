"""The escape histogram of a run in cells where most photons leave by few bins: a slab of 8 voxels,
one bin and the most bins there are, against the histogram of one atomic per visit."""
import pytest
import torch

from paper_2604_13929_amd import inputs, photonmc as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [(1.0, 1), (8.0, 256), (0.05, 512)])
@pytest.mark.parametrize("opt,fp64", [(pm.Optics(0.5, 0.01, 0.7), False), (pm.paper_optics(0.5, 0.01, 0.7, gate=40.0), False),
                                      (pm.Optics(0.5, 0.01, 0.7), True)])
def test_few_bins(bins, opt, fp64):
    mask = inputs.spinodal_mask_torch(320, 250, 8, 12.0, 0.7, seed=4, device=torch.device("cuda:0"))
    n = 4_000_000
    a = pm.run(mask, opt, n, 5, fp64=fp64, escape_bins=bins)
    b = pm.run(mask, opt, n, 5, fp64=fp64, escape_bins=bins, direct=True)
    assert torch.equal(a.fluence, b.fluence) and torch.equal(a.scalars, b.scalars)
    assert torch.equal(a.escape_hist_w, b.escape_hist_w) and torch.equal(a.escape_hist_n, b.escape_hist_n)
    assert int(a.escape_hist_n.sum()) == a.scalar_dict()["esc_n"]
