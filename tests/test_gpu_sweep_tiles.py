"""Bias sweep (Sec. 3.2) over several row tiles, at the class counts where a tile's rows halve (128 to 16
rows of 33 to 256 classes) and at tile counts that the XCDs' runs share unevenly, against numpy
binary64 (exact)."""
import numpy as np
import pytest
import torch

from paper_2409_08270_amd import _lib as L
from tests.test_gpu_rows import _a, _normalised

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,E", [(1291, 33), (1281, 34), (450, 66), (451, 67), (545, 131), (273, 132), (129, 256), (257, 256),
                                 (4097, 17), (16, 256), (1, 256)])
def test_sweep_tile_edges(n, E):
    ctx = L.Context()
    A, lo, dA, dlo = _a(n, E, n, n % 2 == 1)
    gammas = np.linspace(-0.4, 0.6, min(9, 4096 // E)).astype(np.float32)
    with np.errstate(all="ignore"):
        _, _, an, on = _normalised(A, lo)
        want = np.stack([(an > on + np.float64(g)).T for g in gammas])
    S = torch.full((len(gammas), E, n), 7, dtype=torch.uint8, device="cuda")
    assert np.array_equal(ctx.fs_assign_sweep(dA, dlo, n, E, gammas, S), want.sum(2))
    assert np.array_equal(S.cpu().numpy(), want.astype(np.uint8))
