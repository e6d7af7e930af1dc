"""Calls over the first targets of a layout: total_tiles counts tiles that no target of the call owns.  They are empty,
and nothing past the call's targets is written."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("count", [1, 2, 10])
def test_loss_of_the_first_targets(count):
    """The losses and gradients of the first targets are those of the whole call; the others' stay as they were."""
    from paper_2311_16728_amd import gs

    plan = plan_for([scenes.pinhole(150, 110, 80.0)] * 4, levels=(0, 1, 2))
    g = torch.Generator().manual_seed(3)
    plan.rgb.copy_(torch.rand(plan.rgb.shape, generator=g))
    y = torch.rand(plan.rgb.shape, generator=g).cuda()
    plan.loss(y, 0.2, True)
    whole, losses = plan.dL.clone(), plan.d_loss.clone()
    room = torch.full((3 * whole.numel(),), -5.0, device="cuda")   # (the gradient, between two margins)
    dL = room[whole.numel():2 * whole.numel()]
    plan.d_loss.fill_(-5.0)
    gs.gs_pyramid_loss(plan.rgb, y, plan.targets_dev, count, plan.total_tiles, plan.total_pixels, 0.2, plan.loss_ws,
                       plan.d_loss, plan.d_total, dL)
    end = 3 * plan.target_slice(count)[0]
    assert torch.equal(dL[:end], whole[:end]) and torch.equal(plan.d_loss[:count], losses[:count])
    assert torch.all(plan.d_loss[count:] == -5.0)
    assert torch.all(room[:whole.numel()] == -5.0) and torch.all(room[whole.numel() + end:] == -5.0)


@pytest.mark.parametrize("count", [1, 3, 7])
@pytest.mark.parametrize("n,sizes", [(3000, [(150, 110)] * 4), (70000, [(150, 110)] * 4), (3000, [(801, 613), (33, 40), (799, 620)])])
def test_binning_of_the_first_targets(n, sizes, count):
    """Lists, images and gradients of the first targets are those of the whole call, and the other tiles are empty,
    whatever the workspace held (up to 4,096 tiles and more, small and large chunks, one target and several)."""
    from paper_2311_16728_amd import gs

    p = torch.as_tensor(scenes.draw_gaussians(np.random.default_rng(n), n, (-1, -1, 2), (1, 1, 4))).cuda()
    plan = plan_for([scenes.pinhole(w, h, 0.6 * w) for w, h in sizes], levels=(0, 1, 2), n_cap=p.shape[1], pair_cap=1 << 22)
    plan.render(p, n)
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    S, T, cap, o = plan.n_views * plan.n_cap, plan.n_targets * plan.n_cap, plan.pair_cap, up(64)
    for size in (4 * S, 8 * T, 4 * S, 4 * S, 4 * S, 4 * S, 4 * (S + 1), 4 * cap, 4 * cap, 4 * cap, 4 * cap):
        o = up(o + size)
    ranges = lambda: plan.sort_ws[o:o + 8 * plan.total_tiles].view(torch.int32).reshape(-1, 2).clone()  # noqa: E731
    whole, rgb, last = ranges(), plan.rgb.clone(), plan.last.clone()
    dL = torch.rand(plan.rgb.shape, generator=torch.Generator().manual_seed(1)).cuda()
    tile, pix = plan.targets[count].tile_offset, plan.target_slice(count)[0]
    args = (plan.settings, plan.proj_ws, plan.n_cap, plan.n_views, plan.sort_ws, plan.pair_cap, plan.targets_dev, count,
            plan.total_tiles)
    acc = []
    for fill in (0, 0x5a):
        # (sort_ws is laid out for the call's own targets; a query for all of them is at least as large)
        plan.sort_ws.fill_(fill)
        plan.status.zero_()
        plan.rgb.fill_(-5.0)
        gs.gs_bin_sort(plan.settings, plan.proj_ws, n, plan.n_cap, plan.n_views, plan.targets_dev, count, plan.total_tiles,
                       plan.sort_ws, plan.pair_cap, plan.status)
        gs.gs_render_fwd(*args, plan.rgb, plan.T, plan.last, None)
        assert not plan.overflowed()
        counters = plan.sort_ws[:64].view(torch.int32).cpu()
        assert counters[1] == counters[2] == (whole[:tile, 1] - whole[:tile, 0]).sum()
        assert torch.equal(plan.rgb[:3 * pix], rgb[:3 * pix]) and torch.equal(plan.last[:pix], last[:pix])
        assert torch.all(plan.rgb[3 * pix:] == -5.0)
        gs.gs_raster_bwd(*args, plan.T, plan.last, dL, plan.accum_ws)
        acc.append(plan.accum_ws[:36 * S].view(torch.float32).clone())
    assert acc[0].abs().max() > 0 and torch.allclose(*acc, rtol=1e-3, atol=1e-5 * float(acc[0].abs().max()))
