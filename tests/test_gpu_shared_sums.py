"""One scene's views split over two descriptors of a batch that name the same A (Eq. (7) sums over
views): both descriptors' weights add up, whatever the reduction, the number of classes (float64
totals or two-sum) and zero_accumulators, and both assignments see the whole sum."""
import ctypes

import pytest
import torch

import oracle as O
import scenegen as sg
from paper_2409_08270_amd import _lib as L
from tests._parity import assert_A, assert_labels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reduction", [L.FS_RED_AUTO, L.FS_RED_LDS, L.FS_RED_DET])
@pytest.mark.parametrize("E,zero,shift", [(2, 1, 0), (2, 0, 0), (5, 1, 100), (255, 1, 0)])
def test_descriptors_that_share_sums_add_up(reduction, E, zero, shift):
    sc = sg.make_config("C1", n=900, views=4, res=64)
    sc.E = E
    ctx = L.Context()
    ds = L.DeviceScene(sc)
    halves = [ds.view_subset([0, 2]), ds.view_subset([1, 3])]
    # the second descriptor's Gaussians begin `shift` rows into the first's
    arrays = [a[shift:].contiguous() for a in ds.arrays]
    n2 = sc.n - shift
    hi = torch.zeros((sc.n, E), dtype=torch.float32, device="cuda")
    lo = torch.zeros_like(hi)
    S = [torch.zeros((E, n), dtype=torch.uint8, device="cuda") for n in (sc.n, n2)]
    arr = (L.FsScene * 2)()
    cams = [h.cams()[0] for h in halves]
    for i, (h, n, at) in enumerate(((halves[0], sc.n, 0), (halves[1], n2, shift))):
        g = ds.struct() if i == 0 else L.FsGaussians(*[L._ptr(a) for a in arrays], n2)
        arr[i] = L.FsScene(g, ctypes.cast(cams[i], ctypes.POINTER(L.FsCamera)), 2, L._ptr(h.masks), E,
                           L._ptr(hi[at:]), L._ptr(lo[at:]), L._ptr(S[i]), None, 0.0)
    o = L.batch_opts(reduction=reduction, zero_accumulators=zero)
    b = ctypes.c_void_p()
    ctx._check(ctx.L.fs_batch_create(ctx.h, arr, 2, ctypes.byref(L.params()), ctypes.byref(o), ctypes.byref(b)))
    sub = sg.make_config("C1", n=900, views=4, res=64)
    sub.E = E
    for k in ("mx", "my", "mz", "qw", "qx", "qy", "qz", "sx", "sy", "sz", "op"):
        setattr(sub, k, getattr(sub, k)[shift:].copy())
    first = O.solve64(sc, O.params(), views=[0, 2])
    second = O.solve64(sub, O.params(), views=[1, 3])
    A, slack = first["A"].copy(), first["slack"].copy()
    A[shift:] += second["A"]
    slack[shift:] += second["slack"]
    for run in (1, 2):
        ctx._check(ctx.L.fs_batch_run(b))
        got = (hi.double() + lo.double()).cpu().numpy()
        f = 1 if zero else run
        assert_A(got, f * A, f * slack, what=f"run {run}")
        S64, margin = O.assign64(f * A, 0.0)
        assert_labels(S[0].cpu().numpy(), S64, margin, f * A, got)
        assert_labels(S[1].cpu().numpy(), S64[:, shift:], margin[:, shift:], f * A[shift:], got[shift:])
    ctx.L.fs_batch_destroy(b)
