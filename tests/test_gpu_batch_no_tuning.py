"""A batch that walks in cells looks for no launch shape: nothing is timed or stored, and one that
accumulates needs no tune; a batch by the log is tuned as before."""
import ctypes

import pytest
import torch

from paper_2604_13929_amd import inputs, photonmc as pm

pytestmark = pytest.mark.gpu


def _jobs(n, begin=0):
    return [pm.BatchJob(inputs.spinodal_mask_torch(*d, 12.0, 0.7, seed=4, device=torch.device("cuda:0")),
                        pm.Optics(0.5, 0.01, 0.7), n, 9, stream_id=i, photon_begin=begin, reduce=False)
            for i, d in enumerate([(64, 64, 64), (40, 50, 60), (96, 96, 40)])]


def _same(a, b):
    for x, y in zip(a.results, b.results):
        assert torch.equal(x.fluence, y.fluence) and torch.equal(x.scalars, y.scalars)


def test_cells_are_not_tuned(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("PHOTONMC_TUNE_CACHE", str(cache))
    n = 1_000_000
    want = pm.run_batch(_jobs(2 * n), tune=pm.Tune(), line_staging=True)
    _same(pm.run_batch(_jobs(2 * n)), want)
    halves = pm.run_batch(_jobs(n))
    pm.run_batch(_jobs(n, begin=n), accumulate_into=halves)
    _same(halves, want)
    d = pm.McTune()
    pm.load().mc_tune_default(ctypes.byref(d))
    assert pm.autotune_batch(_jobs(n)) == pm.Tune(d.block, d.waves_per_cu, d.chunk, d.refill, d.defer)
    assert not cache.exists()
    b = pm.Batch(_jobs(n), accumulate_into=halves)
    with pytest.raises(pm.McError, match="accumulates"):
        pm._check(pm.load().mc_autotune_batch(ctypes.byref(b.c_jobs), 3, 0, b.ws.data_ptr(), b.ws.numel(), ctypes.byref(d),
                                              pm._stream(b.device)), "mc_autotune_batch")


def test_the_log_is_tuned(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("PHOTONMC_TUNE_CACHE", str(cache))
    small = pm.run_batch(_jobs(2000))
    assert len(cache.read_text().splitlines()) == 1
    _same(small, pm.run_batch(_jobs(2000), tune=pm.Tune()))
    assert len(cache.read_text().splitlines()) == 1
    other = _jobs(20000)
    with pytest.raises(pm.McError, match="accumulates"):
        pm.run_batch(other, accumulate_into=pm.run_batch(other, tune=pm.Tune()))
