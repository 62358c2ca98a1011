"""The tile-listing rule on splats larger than the image: their candidate and
sure columns carry margins of a few ulp of their extent (csrc/fs_tiles.h), against the oracle's test
of every pixel centre. Means lie
up to three standard deviations outside, so that edges of every slope and the tops of the ellipses
cross the image. No GPU is used."""
import numpy as np
import pytest

import oracle as O
from tests.test_tile_rule import rule  # noqa: F401 (fixture)

CASES = [  # W, H, tile, sigma range (px), conditioning bound, float32 path forced
    (640, 480, 16, 16, 100.0, 3e3, 64.0, False),
    (333, 241, 16, 16, 3e3, 1e6, 64.0, False),
    (1297, 840, 32, 8, 300.0, 1e5, 64.0, False),
    (300, 200, 8, 32, 300.0, 1e5, 1e5, True),
]


@pytest.mark.parametrize("case", CASES)
def test_large_splats(rule, case):  # noqa: F811
    W, H, tw, th, smin, smax, cond, force = case
    rng = np.random.default_rng(70 + CASES.index(case))
    n = 6000
    ang = rng.uniform(0, np.pi, n)
    s1 = np.exp(rng.uniform(np.log(smin), np.log(smax), n))
    s2 = np.exp(rng.uniform(np.log(smin * 0.05), np.log(smax), n))
    co, si = np.cos(ang), np.sin(ang)
    # one point of the ellipse near k = 3 lands in the image, so that its edge crosses it
    th0 = rng.uniform(0, 2 * np.pi, n)
    k = 3.0 * (1.0 + rng.choice([0.0, 1e-4, 3e-3, 0.1], n) * rng.normal(size=n))
    ex, ey = k * s1 * np.cos(th0), k * s2 * np.sin(th0)
    u = (rng.uniform(0, W, n) - (co * ex - si * ey)).astype(np.float32)
    v = (rng.uniform(0, H, n) - (si * ex + co * ey)).astype(np.float32)
    a = (co * co * s1 * s1 + si * si * s2 * s2 + 0.3).astype(np.float32)
    b = (co * si * (s1 * s1 - s2 * s2)).astype(np.float32)
    c = (si * si * s1 * s1 + co * co * s2 * s2 + 0.3).astype(np.float32)
    det = (a * c - b * b).astype(np.float32)
    deg = ~(det > 0) | ((a * c).astype(np.float32) >= np.float32(cond) * det)
    flags = np.where(deg & ~np.bool_(force), 3, 1).astype(np.uint8)
    keep = flags == 1
    m, cv, f = np.stack([u, v], 1)[keep], np.stack([a, b, c], 1)[keep], flags[keep]
    rect = np.tile(np.array([0, 0, (W - 1) // tw, (H - 1) // th], np.int32), (len(f), 1))
    rows = (H + th - 1) // th
    got = rule(m, cv, f, rect, tw, th, W, H, rows)
    ref = O.listed_rows32(m, cv, f, rect, tw, th, W, H, max_rows=rows)
    bad = np.nonzero((got != ref).any(axis=(1, 2)))[0]
    assert len(bad) == 0, (len(bad), m[bad[0]], cv[bad[0]], got[bad[0]].tolist(), ref[bad[0]].tolist())
    inside = (ref[:, :, 0] > 0) | ((ref[:, :, 1] >= 0) & (ref[:, :, 1] < (W - 1) // tw))
    assert len(f) > 1000 and inside.any(axis=1).mean() > 0.2  # edges do cross the image
