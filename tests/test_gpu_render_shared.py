"""Novel-view masks (Sec. 3.4) with the waves of a tile sharing the walk over its list, which large
scenes and many objects take: an object's masks do not depend on the other objects, so every object's
rho and depth are compared bit for bit with a call of few objects, where each wave walks by itself.
Lists are longer than what is staged at once, some are empty, pixels stop early, and Gaussians belong
to several objects or to none."""
import numpy as np
import pytest
import torch

import oracle as O
import scenegen as sg
from paper_2409_08270_amd import _lib as L
from tests.test_gpu_render_blocks import _render

pytestmark = pytest.mark.gpu


def _scene(n, W, H, seed, scale):
    rng = np.random.default_rng(seed)
    means = np.concatenate([rng.normal(scale=0.25, size=(n // 2, 3)), rng.uniform(-1.2, 1.2, size=(n - n // 2, 3))])
    scales = np.exp(rng.normal(np.log(scale), 0.6, (n, 3)))
    poses = [sg.look_at((0.0, -4.0, 0.3), (0.0, 0.0, 0.0)), sg.look_at((2.5, -3.0, 1.0), (0.5, 0.0, 0.3))]
    return sg.make_custom(means[rng.permutation(n)], scales, rng.normal(size=(n, 4)), rng.uniform(0.05, 0.99, n), poses,
                          W=W, H=H, masks=[np.zeros((H, W), np.uint8)] * 2, E=2, focal=60.0)


@pytest.mark.parametrize("n,E,mode,tile,exact", [(70000, 256, L.FS_MASK_DEPTH, (16, 16), False),
                                                 (70000, 241, L.FS_MASK_ARGMAX, (8, 32), False),
                                                 (70000, 256, L.FS_MASK_DEPTH, (32, 8), True)])
def test_many_objects(n, E, mode, tile, exact):
    W, H = 77, 45
    sc = _scene(n, W, H, E + mode, 0.02)
    rng = np.random.default_rng(E)
    S = (rng.random((E, n), dtype=np.float32) < 1.2 / E).astype(np.uint8)
    S[3] = 0                                  # an object of no Gaussian
    S[5] = (rng.random(n) < 0.5)              # and one of half of them
    dS = torch.from_numpy(S).cuda()
    ctx = L.Context()
    prm = (L.params_exact if exact else L.params)(tile_w=tile[0], tile_h=tile[1])
    lab, rho, dep = _render(ctx, sc, dS, E, mode, prm)
    e0 = 0 if mode == L.FS_MASK_ARGMAX else 1
    for lo in (e0, 15, 16, 17, 128, E - 15):
        objects = list(range(lo, min(E, lo + 15)))
        few = torch.cat([dS[:1]] * e0 + [dS[objects]]).contiguous()
        _, r, d = _render(ctx, sc, few, len(few), mode, prm)
        assert np.array_equal(rho[objects].view(np.uint32), r[e0:].view(np.uint32)), lo
        assert np.array_equal(dep[objects].view(np.uint32), d[e0:].view(np.uint32)), lo
    if mode == L.FS_MASK_ARGMAX:
        assert np.array_equal(lab, rho.argmax(0).astype(np.uint8))
    else:
        d = np.where(rho > np.float32(0.1), dep, np.float32(3.0e38))
        d[0] = np.float32(3.0e38)
        assert np.array_equal(lab, np.where(d.min(0) < 3.0e38, d.argmin(0), 0).astype(np.uint8))


@pytest.mark.parametrize("n", [400000, 400321])
def test_one_object(n):
    W, H = 66, 50
    sc = _scene(n, W, H, n, 0.01)
    rng = np.random.default_rng(n)
    S = (rng.random((3, n), dtype=np.float32) < 0.1).astype(np.uint8)
    ctx = L.Context()
    dS = torch.from_numpy(S).cuda()
    one = _render(ctx, sc, dS[:2].contiguous(), 2, L.FS_MASK_DEPTH, L.params())
    two = _render(ctx, sc, dS, 3, L.FS_MASK_DEPTH, L.params())
    assert np.array_equal(one[1][1].view(np.uint32), two[1][1].view(np.uint32))
    assert np.array_equal(one[2][1].view(np.uint32), two[2][1].view(np.uint32))


def test_one_walk_of_a_large_scene():
    # 1M Gaussians, 1,056 tiles of 16x16 over two views: shared; one view of them is not
    n, W, H, E = 1000000, 704, 192, 6
    sc = _scene(n, W, H, 3, 0.01)
    rng = np.random.default_rng(9)
    gt = rng.integers(0, E, n)
    S = (gt[None, :] == np.arange(E)[:, None]).astype(np.uint8)
    dS = torch.from_numpy(S).cuda()
    ctx = L.Context()
    both = _render(ctx, sc, dS, E, L.FS_MASK_DEPTH, L.params())
    for v in range(2):
        each = _render(ctx, sc.subset_views([v]), dS, E, L.FS_MASK_DEPTH, L.params())
        px = slice(v * W * H, (v + 1) * W * H)
        assert np.array_equal(both[0][px], each[0])
        for k in (1, 2):
            assert np.array_equal(both[k][1:, px].copy().view(np.uint32), each[k][1:].view(np.uint32))


def test_against_the_oracle():
    n, E, W, H = 63000, 256, 48, 40
    sc = _scene(n, W, H, 11, 0.015)
    rng = np.random.default_rng(11)
    S = (rng.random((E, n), dtype=np.float32) < 2.0 / E).astype(np.uint8)
    ctx = L.Context()
    _, rho, _ = _render(ctx, sc, torch.from_numpy(S).cuda(), E, L.FS_MASK_DEPTH, L.params_exact())
    prm = O.params(alpha_min=0.0, alpha_max=1.0, t_min=0.0)
    for v in range(2):
        _, r64, _ = O.render_masks64(sc, v, prm, S, tau=0.1, mode=0)
        # one threshold decision taken differently moves rho by at most o * exp(-9/2) ~ 0.011 at the
        # support's edge, two in one pixel by twice that
        d = np.abs(rho[1:, v * W * H:(v + 1) * W * H].reshape(-1, H, W) - r64[1:])
        assert np.quantile(d, 0.999) <= 1e-4 and d.max() <= 0.025, (v, float(d.max()))
