"""Compaction at the edges of its 64-, 256- and 1024-Gaussian runs, against the oracle, exactly; none,
all and a share of the Gaussians selected; `select` may be overwritten as soon as the call returns."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2409_08270_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 257, 1023, 1024, 1025, 2048, 70001])
@pytest.mark.parametrize("share", [0.0, 0.3, 1.0])
def test_compact(n, share):
    rng = np.random.default_rng(n)
    arrays = [rng.normal(size=n).astype(np.float32) for _ in range(11)]
    ds = L.DeviceScene.__new__(L.DeviceScene)
    ds.n, ds.arrays = n, [torch.from_numpy(a).cuda() for a in arrays]
    sel = (rng.random(n) < share).astype(np.uint8) * rng.integers(1, 255, n).astype(np.uint8)
    ctx = L.Context()
    for keep in (False, True):
        # an odd start, so that nothing rests on the alignment of `select`
        s = torch.from_numpy(np.concatenate([np.zeros(1, np.uint8), sel])).cuda()[1:]
        got, idx = ctx.fs_compact(ds, s, keep)
        s.fill_(1)
        want, widx = O.compact64(arrays, sel, keep)
        assert np.array_equal(idx[:len(widx)].cpu().numpy(), widx)
        for g, w in zip(got, want):
            assert np.array_equal(g[:len(widx)].cpu().numpy().view(np.uint32), np.asarray(w, np.float32).view(np.uint32))
