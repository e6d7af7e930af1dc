"""Tile lists of primitives of every footprint, from a pixel to the whole image, on images from one window of tiles to
several, against rectangles computed on the host: which tiles a primitive is listed in, and each tile's order."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, proj_records, require_gpu
from tests.test_gpu_overflow import _pairs
from tests.test_gpu_tile_order import _lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _scene(kind, n, aspect, seed=0):
    rng = np.random.default_rng(seed)
    p = scenes.draw_gaussians(rng, n, (-1, -1, 3), (1, 1, 9))
    p[0, :n] *= p[2, :n]
    p[1, :n] *= p[2, :n] * aspect
    p[10, :n] = 0.0
    scale = np.full((3, n), 0.01)
    if kind == "huge":
        scale[:] = 3.0
    elif kind == "needles":
        scale[:] = [[1.0], [0.004], [0.004]]
    elif kind == "tail":   # the large ones are neighbours in the map
        scale[:, n - n // 100:] = 0.5
    p[3:6, :n] = np.log(scale)
    return p


def _edges(plan, ti, n, grow):
    """Pixel rectangles of the records of target ti, every edge moved out by `grow` of its rounding: (x0, x1, y0, y1) in
    tiles, and which records have one."""
    t, s = plan.targets[ti], plan.settings
    mean, cov, _ = proj_records(plan, n)
    at = plan.specs[ti][0] * plan.n_cap + np.arange(n)
    c, sc = cov[at].astype(np.float64), 0.5 ** t.level
    shown = cov[at, 3] >= np.float32(s.alpha_min)
    tq = 2.0 * np.log(np.where(shown, c[:, 3] / np.float32(s.alpha_min), 1.0))
    out = []
    for m, v, size in ((mean[at, 0], c[:, 0], t.width), (mean[at, 1], c[:, 2], t.height)):
        m, e = m * sc, np.sqrt(tq * (v * sc * sc + s.dilation))
        e = e + 0.05 + 1e-3 * e
        e = e + grow * (0.01 + 1e-5 * e)   # (float32 positions below 2^17 and extents)
        a, b = np.ceil(m - e), np.floor(m + e)
        shown &= (b >= 0) & (a <= size - 1) & (a <= b)
        out += [np.clip(a, 0, size - 1) // 16, np.clip(b, 0, size - 1) // 16]
    return [x.astype(np.int64) for x in out], shown


def _codes(plan, ti, n, grow):
    """Codes tile * n + record of the pairs of target ti."""
    (x0, x1, y0, y1), shown = _edges(plan, ti, n, grow)
    tx = plan.targets[ti].tiles_x
    rows = []
    for r in np.flatnonzero(shown):
        tiles = np.arange(y0[r], y1[r] + 1)[:, None] * tx + np.arange(x0[r], x1[r] + 1)
        rows.append(tiles.ravel() * n + r)
    return np.sort(np.concatenate(rows))


# 1,200 tiles; 3,750; 5,175; 17,441 (two windows); a row of 4,375 beside a small target (windows shorter than a row);
# several targets of up to 4,096 tiles in all, of more, and of several windows
SIZES = [[(640, 480)], [(1200, 800)], [(1200, 1100)], [(2600, 1700)], [(70000, 16), (40, 30)], [(900, 700), (600, 400)],
         [(640, 480), (320, 240), (1300, 900)], [(2600, 1700), (1300, 1200)]]


@pytest.mark.parametrize("kind,n", [("small", 1), ("small", 5000), ("huge", 1), ("huge", 300), ("needles", 4000),
                                    ("tail", 30000), ("tail", 140000)])
@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: "+".join("%dx%d" % x for x in s))
def test_lists_hold_every_tile_of_a_footprint(sizes, kind, n):
    w, h = sizes[0]
    p = torch.as_tensor(_scene(kind, n, h / w)).cuda()
    cams = [scenes.pinhole(w, h, 0.5 * w) for w, h in sizes]
    plan = plan_for(cams, n_cap=p.shape[1], pair_cap=1 << 24)
    plan.render(p, n)
    assert not plan.overflowed()
    z = proj_records(plan, n)[2][:, 3]
    for ti in range(plan.n_targets):
        lists = _lists(plan, ti)
        ids = np.concatenate(lists).astype(np.int64)
        tile = np.repeat(np.arange(len(lists)), [len(x) for x in lists])
        depth = z[plan.specs[ti][0] * plan.n_cap + ids]
        assert np.array_equal(np.lexsort((ids, depth, tile)), np.arange(len(ids)))
        got = np.sort(tile * n + ids)
        assert (np.diff(got) > 0).all()
        assert np.isin(_codes(plan, ti, n, -1.0), got, assume_unique=True).all()
        assert np.isin(got, _codes(plan, ti, n, 1.0), assume_unique=True).all()


@pytest.mark.parametrize("sizes", SIZES[1:4] + SIZES[6:], ids=lambda s: "+".join("%dx%d" % x for x in s))
def test_first_pairs_of_large_footprints_are_kept(sizes):
    n, (w, h) = 300, sizes[0]
    p = torch.as_tensor(_scene("huge", n, h / w)).cuda()
    cams = [scenes.pinhole(w, h, 0.5 * w) for w, h in sizes]
    full = plan_for(cams, n_cap=p.shape[1], pair_cap=1 << 24)
    full.render(p, n)
    rows = _pairs(full, n)
    cap = len(rows) // 3
    plan = plan_for(cams, n_cap=p.shape[1], pair_cap=cap)
    plan.render(p, n)
    assert plan.overflowed() and not full.overflowed()
    kept = rows[:cap]
    for ti in range(plan.n_targets):
        mine = kept[kept[:, 2] == ti]
        mine = mine[np.argsort(mine[:, 3], kind="stable")]
        np.testing.assert_array_equal(np.concatenate(_lists(plan, ti)), mine[:, 1] % plan.n_cap)
        np.testing.assert_array_equal([len(x) for x in _lists(plan, ti)],
                                      np.bincount(mine[:, 3], minlength=len(_lists(plan, ti))))


def test_first_pairs_of_many_lists_are_kept():
    """40 targets of 40 chunks: more lists than the items they are shared out in."""
    n = 20000
    p = torch.as_tensor(_scene("small", n, 0.75)).cuda()
    cams = [scenes.pinhole(64 + 8 * (i % 3), 48, 40.0 + i) for i in range(40)]
    full = plan_for(cams, n_cap=p.shape[1], pair_cap=1 << 22)
    full.render(p, n)
    rows = _pairs(full, n)
    cap = len(rows) // 2
    plan = plan_for(cams, n_cap=p.shape[1], pair_cap=cap)
    for _ in range(2):
        plan.render(p, n)
        assert plan.overflowed() and not full.overflowed()
        kept = rows[:cap]
        for ti in range(plan.n_targets):
            mine = kept[kept[:, 2] == ti]
            mine = mine[np.argsort(mine[:, 3], kind="stable")]
            np.testing.assert_array_equal(np.concatenate(_lists(plan, ti)), mine[:, 1] % plan.n_cap)
