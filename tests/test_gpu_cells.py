"""The cell walk of large runs against the deposit log: a run given the workspace it asks for
walks its photons cell by cell; one given the least workspace it accepts (no cell scratch)
logs its deposits.  Both must give the same integers.  Sizes at the edges of cells (32 voxels),
volumes narrower than one, words that wrap (few columns), every boundary model, both transports,
the escape histogram, the gradient bins, step caps, sources and scratch for fewer photons."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2604_13929_amd import inputs, photonmc as pm

pytestmark = pytest.mark.gpu

N = 2_100_000          # the rounds start at 2e6 photons
SEED = 77
PLAIN = pm.Optics(0.5, float(np.float32(0.01)), float(np.float32(0.7)))
PAPER = pm.paper_optics(0.5, float(np.float32(0.01)), float(np.float32(0.7)), gate=600.0)


def _mask(nx, ny, nz, phi=0.7):
    return torch.from_numpy(inputs.spinodal_mask(nx, ny, nz, 12.0, phi, seed=4)).to("cuda:0")


def _bytes(mask, n):
    """The least workspace a run takes, and what it makes use of beyond that."""
    L, vol = pm.load(), pm.volume(mask)
    return L.mc_run_workspace_bytes(ctypes.byref(vol)), L.mc_run_extra_workspace_bytes(ctypes.byref(vol), n)


def _run(mask, opt, n, ws_bytes=None, fp64=False, bins=None, offset=0):
    L = pm.load()
    vol, o = pm.volume(mask), opt.c()
    nbytes = sum(_bytes(mask, n)) if ws_bytes is None else ws_bytes
    ws = torch.empty(nbytes + offset, dtype=torch.uint8, device="cuda:0")
    f = torch.empty(tuple(mask.shape), dtype=torch.int64, device="cuda:0")
    s = torch.empty(pm.NSCALARS, dtype=torch.int64, device="cuda:0")
    flags = pm.MC_FP64 if fp64 else 0
    stream = pm._stream(mask.device)
    ptr = ws.data_ptr() + offset
    if bins is None:
        pm._check(L.mc_run(ctypes.byref(vol), ctypes.byref(o), 5, n, SEED, 3, flags, f.data_ptr(), s.data_ptr(), ptr,
                           nbytes, None, stream), "mc_run")
        torch.cuda.synchronize()
        return f, s
    hw = torch.empty(bins, dtype=torch.int64, device="cuda:0")
    hn = torch.empty(bins, dtype=torch.int64, device="cuda:0")
    pm._check(L.mc_run_escape_histogram(ctypes.byref(vol), ctypes.byref(o), 5, n, SEED, 3, flags, f.data_ptr(),
                                        s.data_ptr(), ptr, nbytes, None, 7.5, bins, hw.data_ptr(), hn.data_ptr(), stream),
              "mc_run_escape_histogram")
    torch.cuda.synchronize()
    return f, s, hw, hn


def _same(a, b):
    for x, y in zip(a, b):
        assert torch.equal(x, y)


CASES = [
    ("one cell", (32, 32, 32), PLAIN, {}),
    ("one voxel over", (33, 33, 33), PLAIN, {}),
    ("ragged", (70, 33, 61), PLAIN, {}),
    ("thin", (1, 65, 40), PLAIN, {}),
    ("hot words", (3, 4, 30), PLAIN, {}),
    ("hot words, pads", (3, 4, 30), PAPER, {}),
    ("mirrors and gate", (40, 31, 62), PAPER, {}),
    ("pads over a cell", (20, 20, 31), PAPER, {}),
    ("periodic Fresnel", (40, 31, 50), pm.paper_optics(0.3, 0.02, 0.5, lateral=pm.LATERAL_PERIODIC), {}),
    ("fp64", (40, 31, 50), PLAIN, dict(fp64=True)),
    ("fp64 mirrors", (31, 20, 40), PAPER, dict(fp64=True)),
    ("histogram", (40, 31, 50), PLAIN, dict(bins=64)),
    ("histogram, mirrors", (31, 20, 40), PAPER, dict(bins=512)),
    ("step cap", (40, 31, 50), pm.Optics(0.5, 0.01, 0.7, max_steps=70), {}),
    ("Lambertian", (40, 31, 50), pm.Optics(0.5, 0.01, 0.7, source=1), {}),
    ("no absorption", (40, 31, 50), pm.Optics(0.5, 0.0, 0.0), {}),
    ("no scattering", (40, 31, 50), pm.Optics(0.0, 0.05, 0.0), {}),
    ("no interaction", (40, 31, 50), pm.Optics(0.0, 0.0, 0.0), {}),
    ("roulette", (40, 31, 50), pm.Optics(0.5, 0.2, 0.7, w_roulette=0.05, roulette_m=4), {}),
    ("path cap", (40, 31, 50), pm.Optics(0.5, 0.01, 0.7, path_cap=60.0), {}),
]


@pytest.mark.parametrize("name,dims,opt,kw", CASES, ids=[c[0] for c in CASES])
def test_cells_equal_log(name, dims, opt, kw):
    mask = _mask(*dims)
    least = _run(mask, opt, N, ws_bytes=_bytes(mask, N)[0], **kw)
    _same(_run(mask, opt, N, **kw), least)
    assert int(least[1][pm.SCALARS.index("launched")]) == N


def test_less_scratch_and_unaligned():
    """Scratch for a quarter of the photons (slots are used again), less than asked for, too little
    to use, and a workspace that starts at 8 bytes."""
    mask = _mask(70, 33, 61)
    least = _run(mask, PLAIN, 2 * N, ws_bytes=_bytes(mask, N)[0])
    need, extra = _bytes(mask, 2 * N)
    assert 72 * N // 3 < extra < 72 * N
    for nbytes in (need + extra, need + extra - (1 << 20), need + (20 << 20)):
        _same(_run(mask, PLAIN, 2 * N, ws_bytes=nbytes, offset=8), least)


@pytest.mark.parametrize("opt,fp64", [(PLAIN, False), (PAPER, False), (PLAIN, True), (PAPER, True)])
def test_gradient_cells_equal_log(opt, fp64):
    mask = _mask(33, 40, 50)
    a = pm.grad(mask, opt, N, SEED, fp64=fp64)
    b = pm.grad(mask, opt, N, SEED, fp64=fp64, line_staging=True)
    value = lambda r: (r.bins[..., 0] << 32) + r.bins[..., 1]
    _same((a.run.fluence, a.run.scalars, value(a)), (b.run.fluence, b.run.scalars, value(b)))


def test_all_solid_and_all_pore():
    for pore in (False, True):
        mask = torch.from_numpy(inputs.homogeneous_mask(34, 30, 40, pore=pore)).to("cuda:0")
        _same(_run(mask, PLAIN, N), _run(mask, PLAIN, N, ws_bytes=_bytes(mask, N)[0]))


@pytest.mark.parametrize("n", [1, 63, 4096, 4097, 100_000, 300_000])
def test_few_photons_spread_over_wavefronts(n):
    """The log walk with fewer photons than lanes (each wavefront takes its share) against one
    atomic per visit with a shape of its own."""
    mask = _mask(40, 31, 50)
    a = pm.run(mask, PLAIN, n, SEED)
    b = pm.run(mask, PLAIN, n, SEED, direct=True, tune=pm.Tune(block=64, waves_per_cu=3, chunk=7, refill=64, defer=64))
    _same((a.fluence, a.scalars), (b.fluence, b.scalars))


def _jobs(paper):
    rng = np.random.default_rng(8)
    jobs = []
    for i, dims in enumerate([(33, 20, 40), (64, 64, 30), (5, 6, 31), (40, 40, 40), (20, 70, 33)]):
        opt = pm.Optics(0.2 + 0.1 * i, 0.01, 0.1 * i)
        if paper and i % 2:
            opt = pm.paper_optics(0.3, 0.01, 0.5, gate=500.0, lateral=i // 2)
        jobs.append(pm.BatchJob(_mask(*dims), opt, int(rng.integers(300_000, 700_000)), SEED, stream_id=i,
                                photon_begin=11 * i, reduce=i != 2))
    return jobs


@pytest.mark.parametrize("paper,fp64,esc", [(False, False, False), (False, False, True), (True, False, True),
                                            (True, True, False)])
def test_batch_cells_equal_log(paper, fp64, esc):
    """Jobs of several cells each, some narrower than one, in one batch of more than 2e6 photons."""
    jobs = _jobs(paper)
    assert sum(j.n_photons for j in jobs) >= 2_000_000
    bins = [(4.0, 50 + i) if i != 1 else None for i in range(len(jobs))] if esc else None
    a = pm.run_batch(jobs, tune=pm.Tune(), fp64=fp64, escape_bins=bins)
    b = pm.run_batch(jobs, tune=pm.Tune(), fp64=fp64, escape_bins=bins, line_staging=True)
    for x, y in zip(a.results, b.results):
        _same((x.fluence, x.scalars), (y.fluence, y.scalars))
        if x.escape_hist_w is not None:
            _same((x.escape_hist_w, x.escape_hist_n), (y.escape_hist_w, y.escape_hist_n))


def test_batch_graph_in_cells():
    """The captured step of a large batch, replayed with eager work in between."""
    jobs = _jobs(False)
    want = pm.run_batch(jobs, tune=pm.Tune(), line_staging=True)
    graph = pm.BatchGraph(jobs, tune=pm.Tune())
    for _ in range(3):
        for r in graph.batch.results:
            r.fluence.fill_(7)
        graph.launch()
        torch.cuda.synchronize()
        for x, y in zip(graph.batch.results, want.results):
            _same((x.fluence, x.scalars), (y.fluence, y.scalars))
    graph.close()
