"""Which pairs a binning keeps that finds more of them than pair_cap: the first in the order (depth, record, target,
row-major in the target), so that every tile keeps its nearest Gaussians, the same ones in every run and whichever of
the two paths the call takes."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, proj_records, require_gpu
from tests.test_gpu_tile_order import _lists, _scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _pairs(plan, n):
    """The call's pairs as rows (depth bits, record, target, tile), in the order in which they are kept."""
    z = proj_records(plan, n)[2][:, 3].view(np.uint32)
    rows = []
    for ti, spec in enumerate(plan.specs):
        for tile, ids in enumerate(_lists(plan, ti)):
            r = ids.astype(np.int64) + spec[0] * plan.n_cap
            rows.append(np.stack([z[r].astype(np.int64), r, np.full_like(r, ti), np.full_like(r, tile)], 1))
    rows = np.concatenate(rows)
    return rows[np.lexsort(rows.T[::-1])]


# (kind, n, cameras, levels): per-tile sorts of small and of large chunks, alone and with several targets, beyond 4,096
# tiles, staged scatter; the record sort (four tiles); a near Gaussian over every tile; equal depths
CASES = [("random", 3000, [(320, 240)], (0,)), ("plane", 3000, [(320, 240), (150, 110)], (0, 1)),
         ("random", 150001, [(645, 470)], (0,)), ("planes", 140000, [(320, 240), (300, 200)], (0, 1, 2)),
         ("random", 20000, [(1200, 900), (1100, 700)], (0, 1)), ("random", 140000, [(1200, 1100)], (0,)),
         ("random", 70000, [(24, 20)], (0,)), ("plane", 70000, [(24, 20)], (0,)), ("near", 2000, [(640, 480)], (0, 1))]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_first_pairs_are_kept(case):
    kind, n, sizes, levels = CASES[case]
    whole = _scene(kind, n)
    if n == 150001:
        whole[3:6] = np.log(0.1)   # (more than 2^21 pairs)
    if kind == "near":
        whole[3:6, ::500] = np.log(3.0)
        whole[2, ::500] = 1.0
    p = torch.as_tensor(whole).cuda()
    cams = [scenes.pinhole(w, h, 0.6 * w) for w, h in sizes]
    full = plan_for(cams, levels, n_cap=p.shape[1], pair_cap=1 << 24)
    full.render(p, n)
    assert not full.overflowed()
    rows = _pairs(full, n)
    need = len(rows)
    assert need == full.pair_count() and need > 1000
    for cap in (1, 777, need // 3, need - 1):
        plan = plan_for(cams, levels, n_cap=p.shape[1], pair_cap=cap)
        got = None
        for run in range(2):
            plan.status.zero_()
            plan.render(p, n)
            assert plan.overflowed()
            counters = plan.sort_ws[:64].view(torch.int32).cpu().numpy()
            assert counters[1] == need and counters[2] == cap
            lists = [_lists(plan, ti) for ti in range(plan.n_targets)]
            if got is None:
                image = plan.rgb.clone()
                got = lists
        assert torch.equal(plan.rgb, image)
        kept = rows[:cap]
        for ti in range(plan.n_targets):
            mine = kept[kept[:, 2] == ti]
            order = np.argsort(mine[:, 3], kind="stable")
            tiles = plan.targets[ti].tiles_x * plan.targets[ti].tiles_y
            want = np.split(mine[order, 1] % plan.n_cap, np.cumsum(np.bincount(mine[:, 3], minlength=tiles))[:-1])
            for a, b, c in zip(lists[ti], want, got[ti]):
                np.testing.assert_array_equal(a, b)
                np.testing.assert_array_equal(a, c)
