"""Point-prompt propagation with several rounds per wave, in the first kernel (many prompts share 16
blocks each: more than 16,384 centres) and in the merge (blocks times k above 256), visited by the
golden section: against the binary32 oracle, exactly, for centres in order of their distance."""
import numpy as np
import pytest

import oracle as O
import scenegen as sg
from paper_2409_08270_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(16385, 5), (33000, 1), (49153, 32), (82000, 3)])
@pytest.mark.parametrize("order", ["random", "falling", "rising"])
def test_rounds(n, k, order):
    rng = np.random.default_rng(n + k)
    means = rng.normal(size=(n, 3))
    if order != "random":
        means = means[np.argsort((-1 if order == "falling" else 1) * np.sum(means ** 2, 1))]
    pose = sg.look_at((0.0, -4.0, 0.5), (0.0, 0.0, 0.0))
    sc = sg.make_custom(means, np.full((n, 3), 0.1), np.tile([1.0, 0, 0, 0], (n, 1)), np.full(n, 0.5), [pose, pose])
    ctx = L.Context()
    ds = L.DeviceScene(sc)
    for count in (1, 64):
        pr = np.stack([rng.uniform(14, 18, count), rng.uniform(14, 18, count), rng.uniform(3.9, 4.1, count)], 1)
        pr = pr.astype(np.float32)
        got = ctx.fs_prompt_propagate(ds, 0, pr, k=k)
        for name, a, b in zip(("chosen", "nearest", "uv", "visible"), got, O.prompt32(sc, 0, pr, k=k)):
            assert np.array_equal(a, b), (name, n, k, order, count)
