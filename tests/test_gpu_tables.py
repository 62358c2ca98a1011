"""The per-call tables and small read-backs: calls in a row without a wait between them reuse the
pinned upload room several times over; more views than it holds go through the staging ring;
results larger than the pinned read-back room come back directly."""
import numpy as np
import pytest
import torch

import scenegen as sg
from paper_2409_08270_amd import _lib as L

pytestmark = pytest.mark.gpu


def _scene(n_views):
    rng = np.random.default_rng(n_views)
    n = 300
    poses = []
    for _ in range(n_views):
        d = rng.normal(size=3)
        poses.append(sg.look_at(tuple(4.0 * d / np.linalg.norm(d)), (0.0, 0.0, 0.0)))
    masks = [np.zeros((16, 24), np.uint8) for _ in poses]
    return sg.make_custom(rng.normal(scale=0.6, size=(n, 3)), np.exp(rng.normal(-2.5, 0.4, size=(n, 3))),
                          rng.normal(size=(n, 4)), rng.uniform(0.2, 0.9, n), poses, W=24, H=16, masks=masks, E=2,
                          focal=30.0)


def test_many_calls_and_many_views():
    V = 700  # 700 view tables are more than the upload room
    sc = _scene(V)
    ctx, ds, prm = L.Context(), L.DeviceScene(sc), L.params()
    cams, nv = ds.cams()
    whole = L.Proj(sc.n, nv)
    ctx.fs_project(ds, cams, nv, prm, whole)
    parts = []
    for v in range(V):
        c, k = ds.cams([v])
        p = L.Proj(sc.n, k)
        ctx.fs_project(ds, c, k, prm, p)
        parts.append(p)
    torch.cuda.synchronize()
    for name in ("rec", "rect", "ntiles", "flags"):
        a = torch.cat([getattr(p, name) for p in parts])
        assert torch.equal(a.view(torch.uint8), getattr(whole, name).view(torch.uint8)), name
    assert int((whole.flags != 0).sum()) > 0


@pytest.mark.parametrize("P", [1, 40])
def test_read_backs(P):
    sc = _scene(250)  # 40 prompts: 90 KB of results, more than the read-back room
    ctx, ds, prm = L.Context(), L.DeviceScene(sc), L.params()
    rng = np.random.default_rng(P)
    pts = np.stack([rng.uniform(0, 24, P), rng.uniform(0, 16, P), rng.uniform(2, 5, P)], 1).astype(np.float32)
    out = ctx.fs_prompt_propagate(ds, 3, pts, 5, prm)
    for i in range(P):
        one = ctx.fs_prompt_propagate(ds, 3, pts[i:i + 1], 5, prm)
        for a, b in zip(out, one):
            assert np.array_equal(a[i:i + 1], b, equal_nan=True)


def test_cameras():
    sc = _scene(3)
    rows = L.DeviceScene(sc).cam_rows
    cams = L.cameras(rows)
    for c, r in zip(cams, np.asarray(rows, np.float32)):
        assert list(c.R) == list(r[:9]) and list(c.t) == list(r[9:12])
        assert (c.fx, c.fy, c.cx, c.cy) == tuple(r[12:16]) and (c.width, c.height) == (24, 16)
    assert len(L.cameras(rows[:0])) == 0
    with pytest.raises((ValueError, OverflowError)):
        L.cameras(np.where(np.arange(18) == 17, np.nan, rows[:1]))
