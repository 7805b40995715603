"""The rank binarisation where its selection changes its way: candidates that just fit and
just do not, ties cut among few and among many equal values, masks at odd addresses."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import cahn_hilliard as och
from paper_2604_13929_amd import photonmc as pm

pytestmark = pytest.mark.gpu

CAP = 8192          # candidates that one workgroup selects from


def _field(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n)
    if kind == "wide":          # every exponent, both signs, infinities
        f = np.ldexp(rng.standard_normal(n), rng.integers(-1000, 1000, n))
        f[:: max(1, n // 5)] = np.inf
        f[1:: max(1, n // 5)] = -np.inf
        return f
    if kind == "few":           # ties of about n / 3 each
        return rng.integers(-1, 2, n).astype(np.float64)
    f = rng.standard_normal(n)  # one value held by exactly `kind` entries, at the rank that is cut
    f[rng.permutation(n)[:kind]] = 0.0
    return f


@pytest.mark.parametrize("n", [15, 16, 33, 1023, 8 * 1024 * 16 - 1, 300_001])
@pytest.mark.parametrize("kind", ["normal", "wide", "few", 14, CAP, CAP + 1])
@pytest.mark.parametrize("offset", [0, 1, 15])
def test_rank_threshold_selection(n, kind, offset):
    if isinstance(kind, int) and kind > n:
        pytest.skip("more ties than entries")
    print(f"n = {n}, field {kind}, mask at +{offset}", flush=True)
    L = pm.load()
    f = _field(kind, n, np.random.default_rng(n + offset))
    below, zero = int((f > 0).sum()), int((f == 0).sum())
    dev = torch.from_numpy(f).cuda()
    buf = torch.full((n + 64,), 7, dtype=torch.uint8, device="cuda")
    ws = pm.workspace(L.mc_rank_threshold_workspace_bytes(n), dev.device)
    for k in {1, n // 2, n - 1, below, below + zero // 2, min(n, below + zero)}:
        buf.fill_(7)
        rc = L.mc_rank_threshold(ctypes.c_void_p(dev.data_ptr()), n, k, ctypes.c_void_p(buf.data_ptr() + offset),
                                 ctypes.c_void_p(ws.data_ptr()), ws.numel(), pm._stream(dev.device))
        assert rc == 0
        got = buf.cpu().numpy()
        want = np.zeros(n, np.uint8)
        want[np.argsort(-(f + 0.0), kind="stable")[:k]] = 1
        assert np.array_equal(got[offset:offset + n], want), k
        assert (got[:offset] == 7).all() and (got[offset + n:] == 7).all()
    assert np.array_equal(och.rank_threshold(f, 0.0), np.zeros(n, np.uint8))
