"""Tile lists longer than one workgroup's sort holds (8,192 pairs), which the per-tile sorts cut into runs over many
workgroups: the lists that the depth sort of the records leaves, for every spread of depths, and images rendered from
them again and again."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, require_gpu
from tests.test_gpu_tile_order import _lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _scene(kind, n, seed=0):
    """n small primitives in front of a camera at the origin."""
    rng = np.random.default_rng(seed)
    p = scenes.draw_gaussians(rng, n, (-1, -1, 20), (1, 1, 24))
    p[3:6] = np.log(0.003)
    z = {"random": rng.uniform(20, 24, n), "plane": np.full(n, 21.0), "wall": rng.uniform(20.0, 20.02, n),
         "planes": 20.0 + rng.integers(0, 3, n), "two": np.where(rng.uniform(size=n) < 0.9, 20.0, rng.uniform(20, 24, n)),
         "sorted": np.linspace(20, 24, n), "saw": 20.0 + 4.0 * (np.arange(n) % 4096) / 4096.0,
         "far": np.where(np.arange(n) % 1000 == 7, 3000.0, rng.uniform(20, 20.5, n))}[kind]
    p[0:2, :n] *= z / 20.0   # (the same pixels whatever the depth)
    p[2, :n] = z
    return p


@pytest.mark.parametrize("kind,n", [(k, n) for k in ("random", "plane", "wall", "planes", "two", "sorted", "saw", "far")
                                    for n in (70000, 300001)] + [("random", 1000000), ("plane", 1000000)])
def test_long_lists_equal_the_record_sort(kind, n):
    """All in one tile, beside a tile of a few and an empty one; alone (more than 16,384 records a tile: the record
    sort) and beside a larger view, whose lists are short, middling and long (the per-tile sorts)."""
    p = torch.as_tensor(_scene(kind, n)).cuda()
    small = scenes.pinhole(40, 30, 20.0, cx=8.0, cy=8.0)
    near = scenes.pinhole(700, 500, 300.0, t=[0.0, 0.0, -15.0])
    wide = scenes.pinhole(1300, 900, 2500.0)
    alone = plan_for([small], n_cap=p.shape[1], pair_cap=2 * n)
    alone.render(p, n)
    assert not alone.overflowed()
    want = _lists(alone, 0)
    assert max(len(x) for x in want) > n // 2
    z = p[2].cpu().numpy()
    for ids in want:
        assert (np.diff(z[ids]) >= 0).all() and all((np.diff(ids) > 0) | (np.diff(z[ids]) > 0))
    # (about 1,900 and 5,200 tiles)
    for cams, at in (([small, near], 0), ([near, wide, small], 2)):
        plan = plan_for(cams, n_cap=p.shape[1], pair_cap=1 << 24)
        for _ in range(3):
            plan.render(p, n)
            assert not plan.overflowed()
            for a, b in zip(_lists(plan, at), want):
                np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n", [8192, 8193, 12288, 12289, 16384, 16385, 20000])
def test_lists_around_a_slice(n):
    """List lengths around one and two slices, by the depths and indices themselves."""
    p = _scene("random", 30000)
    p[2, n:] = -1.0
    z = p[2].copy()
    p = torch.as_tensor(p).cuda()
    plan = plan_for([scenes.pinhole(40, 30, 20.0, cx=8.0, cy=8.0), scenes.pinhole(640, 480, 300.0)], n_cap=p.shape[1])
    plan.render(p, 30000)
    lists = [x for t in range(2) for x in _lists(plan, t)]
    assert max(len(x) for x in lists) == n
    for ids in lists:
        assert len(np.unique(ids)) == len(ids) and (ids < n).all()
        np.testing.assert_array_equal(ids, ids[np.lexsort((ids, z[ids]))])


def test_long_lists_in_a_replayed_graph():
    """Binning of long lists captured once and replayed on other parameters, with eager work in between."""
    n = 200000
    a, b = (torch.as_tensor(_scene(k, n, s)).cuda() for k, s in (("random", 1), ("wall", 2)))
    cams = [scenes.pinhole(40, 30, 20.0, cx=8.0, cy=8.0), scenes.pinhole(700, 500, 300.0, t=[0.0, 0.0, -15.0])]
    plan, eager = (plan_for(cams, n_cap=a.shape[1], pair_cap=1 << 23) for _ in range(2))
    p = a.clone()
    plan.render(p, n)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.render(p, n, stream=torch.cuda.current_stream())
    for q in (a, b, b, a):
        p.copy_(q)
        g.replay()
        eager.render(q, n)
        torch.cuda.synchronize()
        assert torch.equal(plan.rgb, eager.rgb) and torch.equal(plan.last, eager.last)
