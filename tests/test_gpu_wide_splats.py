"""Splats as wide as the image, and tiles that finish early.

Rows of 16 tiles and more are written by a whole wave, 64 tiles at a time, and the later depth slabs
count a splat's tiles from a table of the live ones: image widths around those sizes, with the
bit-reproducible sums, which must not depend on the slabs; the tile lists of one slab against the
oracle's, entry by entry."""
import numpy as np
import pytest
import torch

import scenegen as sg
from paper_2409_08270_amd import _lib as L
from tests._lists import check_chunk_lists

pytestmark = pytest.mark.gpu


def _scene(W, H, seed):
    rng = np.random.default_rng(seed)
    n = 500
    means = rng.normal(scale=0.8, size=(n, 3))
    scales = np.exp(rng.normal(-2.5, 0.5, size=(n, 3)))
    wide = rng.random(n) < 0.3
    scales[wide] = np.exp(rng.normal(0.7, 0.8, size=(int(wide.sum()), 3)))
    thin = rng.random(n) < 0.2
    scales[thin, rng.integers(0, 3, int(thin.sum()))] *= 1e-4
    quats = rng.normal(size=(n, 4))
    op = np.where(rng.random(n) < 0.7, 0.99, rng.random(n))
    poses = [sg.look_at((0.3, -3.5, 0.4), (0.0, 0.0, 0.0)), sg.look_at((2.5, -2.0, 1.5), (0.0, 0.0, 0.0))]
    masks = [rng.integers(0, 3, (H, W)).astype(np.uint8) for _ in poses]
    return sg.make_custom(means, scales, quats, op, poses, W=W, H=H, masks=masks, E=3, focal=0.8 * W)


@pytest.mark.parametrize("W,H,tw,th", [(15, 40, 16, 16), (250, 33, 16, 16), (272, 40, 16, 16), (1024, 20, 16, 16),
                                       (1040, 50, 16, 16), (530, 20, 8, 32), (2080, 24, 32, 8)])
def test_slabs_and_lists(W, H, tw, th):
    sc = _scene(W, H, W + H)
    ctx = L.Context()
    ds = L.DeviceScene(sc)
    prm = L.params(tile_w=tw, tile_h=th)
    want = None
    for slabs in (1, 2, 3, 4):
        b = L.Batch(ctx, [ds], prm, reduction=L.FS_RED_DET, depth_slabs=slabs)
        b.run()
        torch.cuda.synchronize()
        got = (b.A_hi[0].cpu().numpy().view(np.uint32), b.A_lo[0].cpu().numpy().view(np.uint32), b.S[0].cpu().numpy())
        st = ctx.status()
        assert st["flags"] & (L.FS_DEV_PAIR_OVERFLOW | L.FS_DEV_BAD_LABEL) == 0
        if want is None:
            want = got
            pairs = st["pairs_emitted"]
            assert check_chunk_lists(b, [sc], [(0, 0), (0, 1)], prm)[0] == pairs
            ctx.status()
        else:
            assert all(np.array_equal(a, c) for a, c in zip(got, want)), slabs
            assert st["pairs_emitted"] <= pairs
        b.close()
