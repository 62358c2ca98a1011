"""Novel-view masks with a Gaussian whose camera depth overflows to infinity (Sec. 3.4): the depth sums
of the pixels that its support does not reach are those of the scene without it, bit for bit; where it
reaches, the depth is infinite."""
import numpy as np
import pytest
import torch

import scenegen as sg
from paper_2409_08270_amd import _lib as L
from tests.test_gpu_render_blocks import _render

pytestmark = pytest.mark.gpu

W, H = 40, 24


@pytest.mark.parametrize("mode", [L.FS_MASK_DEPTH, L.FS_MASK_ARGMAX])
def test_infinite_depth_stays_in_its_support(mode):
    c = np.float32(np.sqrt(0.5))
    pose = (np.array([[c, 0, -c], [0, 1, 0], [c, 0, c]], np.float32), np.zeros(3, np.float32))
    rng = np.random.default_rng(5)
    n = 60
    cam = np.stack([rng.uniform(-1, 1, n), rng.uniform(-0.6, 0.6, n), rng.uniform(2, 4, n)], 1)
    means = (cam @ pose[0]).astype(np.float32)          # R^T p
    means[-1] = (3e38, 0.0, 3e38)                       # depth 4.2e38: infinite, on the optical axis
    args = dict(W=W, H=H, masks=[np.zeros((H, W), np.uint8)], E=4)
    scales, quats, op = np.full((n, 3), 0.05), rng.normal(size=(n, 4)), rng.uniform(0.4, 0.8, n)
    S = np.zeros((4, n), np.uint8)
    S[rng.integers(0, 4, n), np.arange(n)] = 1
    S[:, -1] = 1                                        # the far one belongs to every object
    ctx, prm = L.Context(), L.params()
    got = _render(ctx, sg.make_custom(means, scales, quats, op, [pose], **args), torch.from_numpy(S).cuda(), 4, mode, prm)
    ref = _render(ctx, sg.make_custom(means[:-1], scales[:-1], quats[:-1], op[:-1], [pose], **args),
                  torch.from_numpy(S[:, :-1].copy()).cuda(), 4, mode, prm)
    dx, dy = np.meshgrid(np.arange(W) + 0.5 - W / 2, np.arange(H) + 0.5 - H / 2)
    away = (dx * dx + dy * dy > 9 * 0.3 + 0.1).reshape(-1)   # support 3 sigma, variance 0.3
    assert np.array_equal(got[0][away], ref[0][away])
    for g, r in zip(got[1:], ref[1:]):
        assert np.array_equal(g[:, away].view(np.uint32), r[:, away].view(np.uint32))
    e0 = 1 if mode == L.FS_MASK_DEPTH else 0
    assert np.all(np.isinf(got[2][e0:, (H // 2) * W + W // 2]))
