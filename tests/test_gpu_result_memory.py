"""What results keep on the device: their outputs and the workspace their call needs, not the extra
scratch of a large run, which a later call has again; results made while that scratch goes round stay right."""
import ctypes

import pytest
import torch

from paper_2604_13929_amd import inputs, photonmc as pm

pytestmark = pytest.mark.gpu

OPT = pm.Optics(0.5, 0.01, 0.7)
N = 2_100_000


def test_results_keep_no_extra_scratch():
    mask = inputs.spinodal_mask_torch(96, 96, 96, 12.0, 0.7, seed=4, device=torch.device("cuda:0"))
    L, vol = pm.load(), pm.volume(mask)
    extra = L.mc_run_extra_workspace_bytes(ctypes.byref(vol), N)
    need = L.mc_grad_workspace_bytes(ctypes.byref(vol)) + (16 << 20)
    assert extra > need
    jobs = [pm.BatchJob(mask, OPT, N, 7, reduce=False)]
    b = pm.Batch(jobs)
    batch_need = L.mc_batch_workspace_bytes(ctypes.byref(b.c_jobs), 1) + mask.numel() * 8 + (1 << 20)
    del b
    for make, most in ((lambda: pm.run(mask, OPT, N, 7), need), (lambda: pm.run(mask, OPT, N, 7, escape_bins=(8.0, 64)), need),
                       (lambda: pm.grad(mask, OPT, N, 7), need), (lambda: pm.run_batch(jobs, tune=pm.Tune()), batch_need)):
        want = make()
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        kept = [make() for _ in range(4)]
        assert torch.cuda.memory_allocated() - before < 4 * most
        torch.cuda.synchronize()
        tally = lambda r: r.results[0].fluence if hasattr(r, "results") else getattr(r, "run", r).fluence
        for r in kept:
            assert torch.equal(tally(r), tally(want))
