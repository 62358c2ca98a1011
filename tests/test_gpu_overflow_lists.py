"""Tile lists of a batch whose inputs grew past the plan.

Every view of a chunk keeps the pairs that fit its planned capacity, in emission order (depth, then
tile), and the excess is dropped and latched. The lists of the other views do not move: they are
compared entry by entry with the oracle's, for the pair sort's one pass (up to 256 tiles a view) and
two passes, with the digit counts scanned and added up by the scatter; the sums of the same run are
compared with the oracle's compositing of those lists."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import scenegen as sg
from paper_2409_08270_amd import _lib as L
from tests._parity import assert_A

pytestmark = pytest.mark.gpu


def _scaled(sc, f):
    f = np.float32(f)
    return dataclasses.replace(sc, sx=sc.sx * f, sy=sc.sy * f, sz=sc.sz * f)


def kept_lists(planned, now):
    """The lists of one chunk that holds every view of the scenes `now` and was planned on `planned`:
    per view its lists (O.bin_view's layout, positions in the chunk), and the number of dropped pairs."""
    prm = O.params()
    views = [(s, v) for s, sc in enumerate(now) for v in range(sc.n_views)]
    plan = [len(O.bin_view(planned[s], v, prm)["g"]) for s, v in views]
    capacity = sum(plan) + sum(plan) // 64 + 4096
    bins = [O.bin_view(now[s], v, prm) for s, v in views]
    ends = np.minimum(np.cumsum([0] + [len(b["g"]) for b in bins]), capacity)
    out, at, dropped = [], 0, max(0, sum(len(b["g"]) for b in bins) - capacity)
    for j, b in enumerate(bins):
        have = int(ends[j + 1] - ends[j])
        keep = min(have, plan[j] + plan[j] // 64 + 256, capacity)
        dropped += have - keep
        rank = np.zeros(len(b["proj"]["depth"]), np.int64)
        rank[np.argsort(b["proj"]["depth"], kind="stable")] = np.arange(rank.size)
        first = np.lexsort((b["tile"], rank[b["g"]]))[:keep]     # emission order
        first = first[np.lexsort((rank[b["g"][first]], b["tile"][first]))]
        n_tiles = b["ranges"].shape[0]
        count = np.bincount(b["tile"][first], minlength=n_tiles)
        start = np.concatenate([[0], np.cumsum(count)[:-1]])
        ranges = np.stack([start, start + count], 1).astype(np.uint32)
        ranges[count == 0] = 0
        out.append(dict(b, g=np.ascontiguousarray(b["g"][first]), tile=b["tile"][first], ranges=ranges, base=at))
        at += keep
    return views, out, dropped


# 36 and 225 tiles take one pass, 324 two; more than 64 block tiles of 4096 pairs in a view go through the scan.
# 1.15 and 1.6: the excess fits the chunk's slack; 2.5 and 4: the chunk overflows too and later views lose pairs
@pytest.mark.parametrize("n,res,grow", [(600, 96, 1.6), (600, 96, 4.0), (600, 288, 1.6), (600, 288, 2.5),
                                        (50000, 240, 1.15), (45000, 288, 1.15)])
def test_lists_past_the_plan(n, res, grow):
    planned = [sg.make_config("C1", seed=s + 1, n=m, views=2, res=res) for s, m in enumerate((n, n + n // 3, n))]
    now = [_scaled(planned[0], grow), planned[1], _scaled(planned[2], 0.1)]
    ctx = L.Context()
    dss = [L.DeviceScene(sc) for sc in planned]
    b = L.Batch(ctx, dss, L.params(), lanes=1)
    ctx.status()
    for ds, sc in zip(dss, now):
        for k, a in zip((7, 8, 9), (sc.sx, sc.sy, sc.sz)):
            ds.arrays[k].copy_(torch.from_numpy(a))
    views, want, dropped = kept_lists(planned, now)
    assert dropped > 0 and b.info()["n_chunks"] == 1
    inf, vals, ranges, refs = b.chunk_lists(0)
    st = ctx.status()
    assert inf["packed"] and refs == views
    assert st["flags"] & L.FS_DEV_PAIR_OVERFLOW and st["pairs_dropped"] == dropped
    t0 = 0
    for (s, v), w in zip(views, want):
        r = ranges[t0:t0 + len(w["ranges"])].astype(np.int64)
        t0 += len(w["ranges"])
        some = w["ranges"][:, 1] > w["ranges"][:, 0]
        assert np.array_equal(r[some], w["ranges"][some].astype(np.int64) + w["base"]), (s, v)
        assert np.all(r[~some] == 0), (s, v)
        assert np.array_equal(vals[w["base"]:w["base"] + len(w["g"])], w["g"]), (s, v)
    b.run()
    prm = O.params()
    for s, sc in enumerate(now):
        A, slack = np.zeros((sc.n, 2)), np.zeros(sc.n)
        for (si, v), w in zip(views, want):
            if si == s:
                # on the binary32 means that the lists are made from: a mean's rounding past
                # pixel 256 alone moves the edge of a splat of lowpass size by 1e-4 of its weight
                p64 = O.project64(sc, v, prm)
                p64[:, 0:2] = w["proj"]["mean2d"]
                O.composite64(sc, v, prm, w, A, slack, p64)
        assert_A((b.A_hi[s].double() + b.A_lo[s].double()).cpu().numpy(), A, slack, what=f"scene {s}")
    b.close()
