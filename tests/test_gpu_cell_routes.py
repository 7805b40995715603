"""Which walk a run takes, seen by what it leaves in the scratch beyond the workspace it needs, and the
walk in cells where MC_CELLS has it taken whatever the size: every model, transport and option at the edges
of cells, against the deposit log, and a run whose rounds end long before its photons are launched."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2604_13929_amd import inputs, photonmc as pm

pytestmark = pytest.mark.gpu

N = 2_100_000
SEED = 77
PLAIN = pm.Optics(0.5, float(np.float32(0.01)), float(np.float32(0.7)))
PAPER = pm.paper_optics(0.5, float(np.float32(0.01)), float(np.float32(0.7)), gate=600.0)
DENSE = pm.Optics(5.0, 0.001, 0.9)
MARK = 0xA5


def _mask(nx, ny, nz, phi=0.7):
    return inputs.spinodal_mask_torch(nx, ny, nz, 12.0, phi, seed=4, device=torch.device("cuda:0"))


def _go(mask, opt, n, flags=0, grad=False, bins=None, extra=None):
    """The results of a run with its extra scratch (or so much of it), and whether it used that scratch."""
    L = pm.load()
    vol, o = pm.volume(mask), opt.c()
    need = (L.mc_grad_workspace_bytes if grad else L.mc_run_workspace_bytes)(ctypes.byref(vol))
    extra = L.mc_run_extra_workspace_bytes(ctypes.byref(vol), n) if extra is None else extra
    ws = torch.full((need + extra,), MARK, dtype=torch.uint8, device="cuda:0")
    f = torch.empty(tuple(mask.shape), dtype=torch.int64, device="cuda:0")
    s = torch.empty(pm.NSCALARS, dtype=torch.int64, device="cuda:0")
    out = [f, s]
    common = (ctypes.byref(vol), ctypes.byref(o), 5, n, SEED, 3, flags, f.data_ptr(), s.data_ptr())
    stream = pm._stream(mask.device)
    if grad:
        b = torch.empty((3, 2, mask.shape[0], 2), dtype=torch.int64, device="cuda:0")
        pm._check(L.mc_grad(*common, b.data_ptr(), None, None, None, ws.data_ptr(), ws.numel(), None, stream), "mc_grad")
        out.append((b[..., 0] << 32) + b[..., 1])
    elif bins:
        hw, hn = (torch.empty(bins, dtype=torch.int64, device="cuda:0") for _ in range(2))
        pm._check(L.mc_run_escape_histogram(*common, ws.data_ptr(), ws.numel(), None, 7.5, bins, hw.data_ptr(), hn.data_ptr(),
                                            stream), "mc_run_escape_histogram")
        out += [hw, hn]
    else:
        pm._check(L.mc_run(*common, ws.data_ptr(), ws.numel(), None, stream), "mc_run")
    torch.cuda.synchronize()
    return out, bool((ws[need:] != MARK).any())


def _same(a, b):
    for x, y in zip(a, b):
        assert torch.equal(x, y)


EDGES = [((32, 32, 32), PLAIN, {}), ((33, 33, 33), PLAIN, {}), ((70, 33, 61), PLAIN, {}), ((1, 65, 40), PLAIN, {}),
         ((3, 4, 30), PLAIN, {}), ((3, 4, 30), PAPER, {}), ((40, 31, 62), PAPER, {}), ((20, 20, 31), PAPER, {}),
         ((40, 31, 50), pm.paper_optics(0.3, 0.02, 0.5, lateral=pm.LATERAL_PERIODIC), {}),
         ((40, 31, 50), PLAIN, dict(flags=pm.MC_FP64)), ((1, 40, 70), PLAIN, dict(flags=pm.MC_FP64)),
         ((31, 20, 40), PAPER, dict(flags=pm.MC_FP64)), ((40, 31, 50), PLAIN, dict(bins=64)),
         ((31, 20, 40), PAPER, dict(bins=512)), ((33, 40, 50), PLAIN, dict(bins=3, flags=pm.MC_FP64)),
         ((33, 40, 50), PLAIN, dict(grad=True)), ((33, 40, 50), PAPER, dict(grad=True)),
         ((33, 40, 50), PLAIN, dict(grad=True, flags=pm.MC_FP64)), ((1, 40, 70), PAPER, dict(grad=True, flags=pm.MC_FP64)),
         ((40, 31, 50), pm.Optics(0.5, 0.01, 0.7, max_steps=70), {}), ((40, 31, 50), pm.Optics(0.5, 0.01, 0.7, source=1), {}),
         ((64, 64, 64), DENSE, {}), ((40, 31, 50), pm.Optics(0.0, 0.05, 0.0), {}), ((40, 31, 50), pm.Optics(0.0, 0.0, 0.0), {}),
         ((40, 31, 50), pm.Optics(0.5, 0.5, 0.7, w_roulette=0.05, roulette_m=4), {})]


@pytest.mark.parametrize("dims,opt,kw", EDGES)
def test_cells_wherever_they_can(dims, opt, kw):
    mask = _mask(*dims)
    log, used = _go(mask, opt, N, extra=0, **kw)
    assert not used
    cells, used = _go(mask, opt, N, **{**kw, "flags": kw.get("flags", 0) | pm.MC_CELLS})
    assert used
    _same(cells, log)


@pytest.mark.parametrize("dims,opt,n,kw,want", [
    ((128, 128, 128), PLAIN, N, {}, True),
    ((128, 128, 128), PLAIN, N, dict(bins=8), True),
    ((128, 128, 128), PLAIN, 1_999_999, {}, False),
    ((128, 128, 128), PLAIN, N, dict(flags=pm.MC_LINE_STAGING), False),
    ((128, 128, 128), PLAIN, N, dict(flags=pm.MC_DIRECT_DEPOSIT | pm.MC_CELLS), False),
    ((128, 128, 128), pm.Optics(0.5, 0.01, 0.7, path_cap=60.0), N, dict(flags=pm.MC_CELLS), False),
    ((128, 128, 128), PLAIN, N, dict(flags=pm.MC_FP64), True),
    ((128, 128, 128), PAPER, N, {}, True),
    ((128, 128, 128), PLAIN, N, dict(grad=True), False),
    ((256, 256, 256), PLAIN, 3 * N, dict(grad=True), True),
    ((256, 256, 256), DENSE, N, {}, False),
    ((320, 320, 8), PLAIN, N, {}, False),
    ((1, 300, 300), PAPER, N, {}, False)])
def test_route(dims, opt, n, kw, want):
    mask = _mask(*dims)
    extra = pm.load().mc_run_extra_workspace_bytes(ctypes.byref(pm.volume(mask)), max(n, N))
    _, used = _go(mask, opt, n, extra=extra, **kw)
    assert used == want


@pytest.mark.parametrize("paper,fp64", [(False, False), (True, False), (True, True)])
def test_batch_in_cells(paper, fp64):
    L = pm.load()
    jobs = [pm.BatchJob(_mask(*d), PAPER if paper and i % 2 else pm.Optics(0.2 + 0.1 * i, 0.01, 0.1 * i), 500_000 + 70_000 * i,
                        SEED, stream_id=i, photon_begin=11 * i)
            for i, d in enumerate([(33, 20, 40), (64, 64, 30), (5, 6, 31), (40, 40, 40)])]
    want = pm.run_batch(jobs, tune=pm.Tune(), fp64=fp64, line_staging=True)
    b = pm.Batch(jobs)
    need = L.mc_batch_workspace_bytes(ctypes.byref(b.c_jobs), len(jobs))
    ws = torch.full_like(b.ws, MARK)
    assert ws.numel() > need
    pm._check(L.mc_run_batch(ctypes.byref(b.c_jobs), len(jobs), pm.MC_CELLS | (pm.MC_FP64 if fp64 else 0),
                             ctypes.byref(pm.Tune().c()), ws.data_ptr(), ws.numel(), pm._stream(b.device)), "mc_run_batch")
    torch.cuda.synchronize()
    assert bool((ws[need:] != MARK).any())
    for x, y in zip(b.results, want.results):
        _same((x.fluence, x.scalars), (y.fluence, y.scalars))


@pytest.mark.parametrize("opt,flags", [(PLAIN, 0), (PAPER, 0), (PLAIN, pm.MC_FP64)])
def test_rounds_end_before_all_are_launched(opt, flags):
    """Scratch for 16000 photons: the rounds enqueued (4000 at most) see some 40 % of the photons launched,
    and the tail takes the others."""
    mask = _mask(64, 64, 512)
    vol = pm.volume(mask)
    # 2 x 2 x 17 cells with the layers of air; what is asked for holds 72 bytes a photon for 24576 a cell
    tables = pm.load().mc_run_extra_workspace_bytes(ctypes.byref(vol), N) - 72 * 24576 * 68
    assert 0 < tables < 1 << 20
    few, used = _go(mask, opt, N, flags=flags | pm.MC_CELLS, extra=tables + 72 * 16000)
    assert used
    _same(few, _go(mask, opt, N, flags=flags, extra=0)[0])
