"""Tile lists of the binning's two paths: by per-tile sorts and by a depth sort of the records.

A target alone takes the record sort when its tiles are few for the number of Gaussians; beside a second, larger
target of another view the call takes the tile sort.  Both must leave the target with exactly the same list in every
tile, whatever the lists' lengths (empty, within the small sort, within the large one, beyond both), with equal
depths, and on maps that fill one tile."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _lists(plan, target):
    """Gaussian indices and ranges of the tiles of one target."""
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    S, T, cap, o = plan.n_views * plan.n_cap, plan.n_targets * plan.n_cap, plan.pair_cap, up(64)
    for size in (4 * S, 8 * T, 4 * S, 4 * S, 4 * S, 4 * S, 4 * (S + 1), 4 * cap, 4 * cap):
        o = up(o + size)
    bits = int(np.ceil(np.log2(plan.total_tiles)))
    second = plan.total_tiles <= 4096 or min((bits + 7) // 8, (bits + 8) // 9) % 2 == 1
    vals = o + (up(4 * cap) if second else 0)
    ranges = o + 2 * up(4 * cap)
    t = plan.targets[target]
    r = plan.sort_ws[ranges:ranges + 8 * plan.total_tiles].view(torch.int32).cpu().numpy().reshape(-1, 2)
    v = plan.sort_ws[vals:vals + 4 * cap].view(torch.int32).cpu().numpy()
    rows = r[t.tile_offset:t.tile_offset + t.tiles_x * t.tiles_y]
    return [v[a:b] % plan.n_cap for a, b in rows]


def _scene(kind, n, total=0, seed=0):
    """Raw parameters of n primitives in front of a camera at the origin, and more behind it up to total."""
    rng = np.random.default_rng(seed)
    p = scenes.draw_gaussians(rng, max(n, total), (-1, -1, 2), (1, 1, 4))
    p[2, n:] = -3.0
    if kind == "plane":      # equal depths: order by index
        p[2, :n] = 3.0
    elif kind == "planes":   # a few depths, each of many primitives
        p[2, :n] = 2.0 + rng.integers(0, 5, n) * 0.25
    elif kind == "far":      # one primitive far behind the others: the depths crowd at one end of the range
        p[2, n - 1] = 4000.0
    elif kind == "copies":
        p[:, n // 2:2 * (n // 2)] = p[:, :n // 2]
    return p


@pytest.mark.parametrize("kind,n", [("random", 1), ("random", 511), ("random", 2047), ("random", 2049), ("random", 5000),
                                    ("random", 8192), ("random", 8193), ("random", 40000), ("plane", 1000),
                                    ("plane", 5000), ("plane", 20000), ("planes", 30000), ("far", 3000), ("far", 9000),
                                    ("copies", 6000), ("random", 0), ("random", 131073)])
def test_paths_leave_the_same_lists(kind, n):
    n_cap = max(n, 70000) // 64 * 64 + 64
    p = torch.zeros(59, n_cap, device="cuda")
    n_cap, whole = p.shape[1], _scene(kind, n, 70000)
    n = max(n, 70000)
    p[:, :n] = torch.as_tensor(whole[:, :n])
    small = scenes.pinhole(24, 20, 20.0)     # four tiles, most primitives in each: alone, the record sort
    large = scenes.pinhole(640, 480, 20.0)   # 1,200 tiles
    # (levels 0 and 1 of the large view: lists of one view's targets and 1,500 tiles; a 1,200 x 1,200 view: 5,625)
    alone = plan_for([small], n_cap=n_cap, pair_cap=1 << 20)
    huge = scenes.pinhole(1200, 1200, 30.0)
    plans = [plan_for([small, large], n_cap=n_cap, pair_cap=1 << 21), plan_for([large, small], (0, 1), n_cap=n_cap,
                                                                               pair_cap=1 << 21),
             plan_for([huge, small], n_cap=n_cap, pair_cap=1 << 22)]
    alone.render(p, n)
    want = _lists(alone, 0)
    image, last = alone.rgb.clone(), alone.last.clone()
    z = p[2].cpu().numpy()
    for ids in want:
        key = list(zip(z[ids], ids))
        assert key == sorted(key)
    for plan, target in zip(plans, (0, 2, 1)):
        plan.render(p, n)
        assert not plan.overflowed()
        got = _lists(plan, target)
        assert len(got) == len(want)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
        assert torch.equal(plan.image(plan.rgb, target).reshape(-1), image)
        assert torch.equal(plan.plane(plan.last, target).reshape(-1), last)


def test_target_of_no_view_is_empty():
    """A target whose view index is outside the call's views has no pairs, beside one that has."""
    p = torch.as_tensor(_scene("random", 3000)).cuda()
    cams = [scenes.pinhole(64, 48, 50.0), scenes.pinhole(80, 64, 60.0)]
    for count in (1, 2):
        plan = plan_for(cams[:count], n_cap=p.shape[1], pair_cap=1 << 18)
        plan.render(p, 3000)
        before = [len(x) for t in range(count) for x in _lists(plan, t)]
        assert sum(before) > 0
        raw = plan.targets_dev.view(torch.int32)
        words = raw.numel() // plan.n_targets
        raw[(count - 1) * words] = 7   # the last target's view
        plan.bin_sort(3000)
        torch.cuda.synchronize()
        assert all(len(x) == 0 for x in _lists(plan, count - 1))
        if count == 2:
            assert [len(x) for x in _lists(plan, 0)] == before[:len(_lists(plan, 0))]


@pytest.mark.parametrize("cap", [1, 63, 1000])
def test_pair_overflow_keeps_the_first_slots(cap):
    """Fewer pair slots than pairs: the flag is raised, the counters hold both numbers and no range passes the end."""
    p = torch.as_tensor(_scene("random", 4000)).cuda()
    plan = plan_for([scenes.pinhole(320, 240, 250.0)], n_cap=p.shape[1], pair_cap=cap)
    plan.render(p, 4000)
    torch.cuda.synchronize()
    counters = plan.sort_ws[:64].view(torch.int32).cpu().numpy()
    assert plan.overflowed() and counters[1] > cap and counters[2] == cap
    assert sum(len(x) for x in _lists(plan, 0)) == cap
    assert torch.isfinite(plan.rgb).all()


@pytest.mark.parametrize("n,big,cap", [(150001, 0, 1 << 23), (150001, 1500, 1 << 23), (262145, 0, 1 << 23), (150001, 0, 1 << 20)])
def test_pairs_staged_by_tile(n, big, cap):
    """One target of more than 2^21 pairs, whose chunks place their pairs by tile in LDS (the first chunks, of large
    primitives, hold more pairs than fit there), beside the same target in a call of two, whose chunks do not."""
    whole = _scene("random", n)
    whole[3:6] = np.log(0.1)
    whole[3:6, :big] = np.log(0.4)
    whole[10] = 0.0
    p = torch.as_tensor(whole).cuda()
    cam = scenes.pinhole(645, 470, 300.0)   # (partial tiles at both edges)
    alone = plan_for([cam], n_cap=p.shape[1], pair_cap=cap)
    beside = plan_for([cam, scenes.pinhole(24, 20, 20.0)], n_cap=p.shape[1], pair_cap=1 << 24)
    alone.render(p, n)
    beside.render(p, n)
    got, want = _lists(alone, 0), _lists(beside, 0)
    assert sum(len(x) for x in want) > 1 << 21 and not beside.overflowed()
    if cap > 1 << 21:
        assert not alone.overflowed()
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
        assert torch.equal(alone.rgb.reshape(-1), beside.image(beside.rgb, 0).reshape(-1))
    else:   # as many as there are slots, those of the last tile in no particular choice
        assert alone.overflowed() and sum(len(x) for x in got) == cap
        for a, b in zip(got, want):
            if len(a) == len(b):
                np.testing.assert_array_equal(a, b)
