"""Which way FS_RED_LDS2SUM sums on either side of 8 sums per pixel, by what each way leaves: float64
totals give A_hi the float nearest to every sum (A zeroed, one call), and a batch holds 8 bytes a sum
for them; the two-sum leaves stray labels' weights in A_lo."""
import numpy as np
import pytest
import torch

from paper_2409_08270_amd import _lib as L
from paper_2409_08270_amd.solve import Solver
from tests.test_gpu_wide import N, VIEWS, _scene

pytestmark = pytest.mark.gpu


def _nearest(hi, lo):
    return np.array_equal((hi.double() + lo.double()).float().cpu().numpy(), hi.cpu().numpy())


@pytest.mark.parametrize("E,totals", [(3, True), (147, True), (148, False)])
def test_modes(E, totals):
    ctx = L.Context()
    ds = L.DeviceScene(_scene(E))
    hi = torch.zeros((N, E), dtype=torch.float32, device="cuda")
    lo = torch.zeros_like(hi)
    Solver(ctx, ds, L.params()).accumulate_views(range(VIEWS), hi, lo)
    assert _nearest(hi, lo) == totals
    b = L.Batch(ctx, [ds], L.params())
    plain = L.Batch(ctx, [ds], L.params(), reduction=L.FS_RED_LDS)
    b.run()
    assert _nearest(b.A_hi[0], b.A_lo[0]) == totals
    extra = b.info()["workspace_bytes"] - plain.info()["workspace_bytes"]
    assert extra == (N * E * 8 if totals else 0)
    # fs_accumulate_noalloc: the two-sum
    h2 = torch.zeros_like(hi)
    l2 = torch.zeros_like(hi)
    s = Solver(ctx, ds, L.params())
    s.accumulate_views(range(VIEWS), h2, l2)
    cams, nv = ds.cams()
    h2.zero_()
    l2.zero_()
    ctx.fs_accumulate_noalloc(s.proj, s.bins, cams, ds.masks, E, L.params(), h2, l2)
    assert not _nearest(h2, l2)
    b.close()
    plain.close()
