"""Point-prompt propagation: the k-lists kept across the lanes of a wave, at the edges of a wave,
of a block's share of the centres and of the number of blocks, against the binary32 oracle
(exact). Centres in falling distance order make every centre an insertion; equal centres tie."""
import numpy as np
import pytest

import oracle as O
import scenegen as sg
from paper_2409_08270_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1025, 5000])
@pytest.mark.parametrize("k", [1, 31, 32])
@pytest.mark.parametrize("order", ["random", "falling", "equal"])
def test_lists(n, k, order):
    rng = np.random.default_rng(n + k)
    means = rng.normal(size=(n, 3))
    if order == "falling":
        means = means[np.argsort(-np.sum(means ** 2, 1))]
    if order == "equal":
        means = np.repeat(means[: max(1, n // 50)], 50, 0)[:n]
        means = np.concatenate([means, np.tile(means[-1:], (n - len(means), 1))])
    pose = sg.look_at((0.0, -4.0, 0.5), (0.0, 0.0, 0.0))
    sc = sg.make_custom(means, np.full((n, 3), 0.1), np.tile([1.0, 0, 0, 0], (n, 1)), np.full(n, 0.5), [pose, pose])
    ctx = L.Context()
    ds = L.DeviceScene(sc)
    for count in (1, 70):
        pr = np.stack([rng.uniform(10, 22, count), rng.uniform(10, 22, count), rng.uniform(3.0, 5.0, count)], 1)
        pr = pr.astype(np.float32)
        got = ctx.fs_prompt_propagate(ds, 0, pr, k=k)
        for name, a, b in zip(("chosen", "nearest", "uv", "visible"), got, O.prompt32(sc, 0, pr, k=k)):
            assert np.array_equal(a, b), (name, n, k, order, count)
