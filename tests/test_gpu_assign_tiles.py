"""Assignment (Sec. 3.2) at the edges of its row tiles: 64 to 512 rows by the number of rows, and the
class counts on either side of the LDS limit, against numpy binary64 (exact)."""
import numpy as np
import pytest
import torch

from paper_2409_08270_amd import _lib as L
from tests.test_gpu_rows import _a, _normalised

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,E", [(524287, 2), (524288, 2), (524289, 2), (525000, 5), (524801, 6), (65535, 2), (65536, 3),
                                 (32767, 4), (16385, 9), (65537, 19), (65600, 20), (66000, 39), (3001, 40), (2007, 77),
                                 (2006, 78)])
def test_tile_edges(n, E):
    ctx = L.Context()
    A, lo, dA, dlo = _a(n, E, n, n % 2 == 1)
    S = torch.full((E, n), 7, dtype=torch.uint8, device="cuda")
    m = torch.full((E, n), 7.0, dtype=torch.float32, device="cuda")
    g = np.float64(np.float32(0.1))
    with np.errstate(all="ignore"):
        v, tot, an, on = _normalised(A, lo)
        want, margin = (an > on + g).T, np.abs(an - on - g).T
        ctx.status()
        ctx.fs_assign(dA, dlo, n, E, 0.1, S, m)
    assert np.array_equal(S.cpu().numpy(), want.astype(np.uint8))
    assert np.array_equal(m.cpu().numpy(), margin.astype(np.float32), equal_nan=True)
    st = ctx.status()
    assert st["unseen"] == int((tot == 0.0).sum())
    assert st["multi_member"] == int((want.sum(0) > 1).sum())
    with np.errstate(invalid="ignore"):
        assert st["low_margin"] == int((margin < 1e-4).sum())
