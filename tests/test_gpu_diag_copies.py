"""Diagnostics (Sec. 4.8) with 1, 2, 4 and 8 copies of the histograms, by rows and classes, against the
oracle's counts (exact)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2409_08270_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,E", [(1, 2), (300, 2), (5000, 256), (700, 100), (5001, 17), (20000, 33), (60001, 17),
                                 (40000, 64)])
def test_copies(n, E):
    rng = np.random.default_rng(n + E)
    A = np.where(rng.random((n, E)) < 0.2, rng.random((n, E)), 0.0).astype(np.float32)
    S = (rng.random((E, n)) < 1.5 / E).astype(np.uint8)
    gt = rng.integers(-1, E + 1, n).astype(np.int32)
    ctx = L.Context()
    dA, dS, dg = (torch.from_numpy(a).cuda() for a in (A, S, gt))
    c, m, o = ctx.fs_diagnose(dA, None, dS, dg, n, E, 0.05)
    ref = O.diagnose64(A.astype(np.float64), S, gt, float(np.float32(0.05)))
    for got, want in zip((c, m, o), ref):
        assert np.array_equal(got.astype(np.int64), np.asarray(want, np.int64))
