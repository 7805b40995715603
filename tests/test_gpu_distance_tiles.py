"""The distance transform at the edges of its packed words and tiles, with sparse solids
(words without any, lines that stay open) and dense ones."""
import numpy as np
import pytest
import torch

from oracle import analytics as oan
from paper_2604_13929_amd import analytics as an

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 2, 31, 32, 33, 63, 64, 65, 97])
@pytest.mark.parametrize("ny,nz", [(3, 5), (512, 2), (513, 2), (1025, 2), (2049, 3), (2, 512), (3, 2049)])
@pytest.mark.parametrize("solid", [2e-4, 0.01, 0.3])
def test_pore_distance_tiles(nx, ny, nz, solid):
    print(f"{nx} x {ny} x {nz}, solid {solid}", flush=True)
    rng = np.random.default_rng(nx * 7 + ny + nz)
    m = (rng.random((nz, ny, nx)) >= solid).astype(np.uint8)
    m.flat[m.size // 2] = 0
    got = an.pore_distance(torch.from_numpy(m).cuda()).cpu().numpy()
    assert np.array_equal(got, oan.pore_distance(m))
