"""fs_accumulate calls that overlap in time on one A (two contexts on two streams, views shared out
between them): every call's weights arrive, in each reduction that adds with atomics. n is small, so
that the calls of both streams keep writing the same entries."""
import pytest
import torch

import oracle as O
import scenegen as sg
from paper_2409_08270_amd import _lib as L
from paper_2409_08270_amd.solve import tiles_of
from tests._parity import assert_A

pytestmark = pytest.mark.gpu

CALLS = 50


@pytest.mark.parametrize("reduction", [L.FS_RED_LDS2SUM, L.FS_RED_LDS, L.FS_RED_PLAIN])
def test_two_streams_add_into_one_a(reduction):
    sc = sg.make_config("C1", n=1000, views=2, res=64)
    ds, prm = L.DeviceScene(sc), L.params()
    hi = torch.zeros((sc.n, 2), dtype=torch.float32, device="cuda")
    lo = torch.zeros_like(hi) if reduction == L.FS_RED_LDS2SUM else None
    torch.cuda.synchronize()
    lanes = []
    for v in range(2):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ctx = L.Context(stream)
            cams, nv = ds.cams([v])
            proj, tiles = L.Proj(sc.n, nv), tiles_of(64, 64, prm)
            ctx.fs_project(ds, cams, nv, prm, proj)
            bins = L.Bins(65536, tiles)
            assert ctx.fs_bin_sort(proj, cams, prm, bins) > 0
            lanes.append((ctx, proj, bins, cams, ds.masks_of(v, v + 1)))
    torch.cuda.synchronize()
    for _ in range(CALLS):
        for ctx, proj, bins, cams, masks in lanes:
            ctx.fs_accumulate(proj, bins, cams, masks, 2, prm, hi, lo, reduction)
    torch.cuda.synchronize()
    ref = O.solve64(sc, O.params())
    A = hi.double() if lo is None else hi.double() + lo.double()
    assert_A(A.cpu().numpy(), CALLS * ref["A"], CALLS * ref["slack"], what=f"reduction {reduction}")
