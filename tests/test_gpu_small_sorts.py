"""Sorts of few items: a single launch up to one block tile (4096 items), and the counts of up to 64
block tiles added up by the scatter itself. Depths repeat, so that the order among equal keys shows.
The lists are compared with the oracle's entry by entry, for one view and for three."""
import numpy as np
import pytest

import scenegen as sg
from paper_2409_08270_amd import _lib as L
from tests._lists import check_chunk_lists
from tests.test_gpu_edges import _check_bins

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    rng = np.random.default_rng(seed)
    # all emit one tile or a few: small splats in front of a camera that looks down the y axis
    means = np.stack([rng.uniform(-1, 1, n), rng.integers(0, max(2, n // 7), n) / max(2, n // 7), rng.uniform(-1, 1, n)], 1)
    scales = np.full((n, 3), 0.004)
    quats = rng.normal(size=(n, 4))
    op = rng.uniform(0.3, 0.95, n)
    poses = [sg.look_at((0.0, -4.0, 0.0), (0.0, 0.0, 0.0)), sg.look_at((0.4, -4.0, 0.3), (0.0, 0.0, 0.0)),
             sg.look_at((-0.4, -4.5, 0.3), (0.0, 0.0, 0.0))]
    masks = [rng.integers(0, 2, (48, 64)).astype(np.uint8) for _ in poses]
    return sg.make_custom(means, scales, quats, op, poses, W=64, H=48, masks=masks, E=2, focal=90.0)


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 1025, 3000, 3600, 4095, 4096, 4097, 8193, 262144, 262145])
def test_small_sorts(n):
    sc = _scene(n, n)
    ctx = L.Context()
    prm = L.params()
    _check_bins(ctx, sc, prm, [0])
    _check_bins(ctx, sc, prm, [0, 1, 2])
    b = L.Batch(ctx, [L.DeviceScene(sc)], prm)
    b.run()
    assert check_chunk_lists(b, [sc], [(0, v) for v in range(3)], prm)[0] > 0
    b.close()
