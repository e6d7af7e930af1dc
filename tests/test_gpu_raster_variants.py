"""Raster variants that only some calls reach: the queued forward with two waves a tile (more than 16,384 tiles), and
the storing variant's backward with one, two and four waves."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import check_gradients, plan_for, require_gpu
from tests.test_gpu_storeall import _cases, _dev, _store_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("views", [8, 7])
def test_queued_forward_of_many_tiles(views):
    """18,000 and 15,750 tiles (either side of the line between two and four waves) from the queue, against the count
    variant: the same bits."""
    from paper_2311_16728_amd.gs import default_settings

    n = 2500
    p, _, _ = scenes.tiny_scene(3, n=n)
    p = _dev(p)
    cams = [scenes.pinhole(800, 720, 500.0 + 20 * v, t=[0.05 * v, 0.0, 0.1], bg=(0.1, 0.2, 0.3)) for v in range(views)]
    plan = plan_for(cams, n_cap=p.shape[1], pair_cap=1 << 22, settings=default_settings(schedule=1))
    assert plan.total_tiles == 2250 * views
    plan.render(p, n)
    assert not plan.overflowed()
    got = [x.clone() for x in (plan.rgb, plan.T, plan.last)]
    for x in (plan.rgb, plan.T):
        x.fill_(float("nan"))
    plan.last.fill_(-7)
    plan.render_fwd(with_ncontrib=True)
    for a, b in zip(got, (plan.rgb, plan.T, plan.last)):
        assert torch.equal(a, b)
    assert all((plan.plane(plan.ncontrib, v) > 0).any() for v in range(views))


@pytest.mark.parametrize("case", ["tiny", "degenerate"])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_stored_backward_with_every_wave_count(orc, case, waves):
    """The stored backward against the oracle, with the metric and bounds of its test at the plans' own wave count."""
    from paper_2311_16728_amd import gs

    name, p, n, cam = [c for c in _cases() if c[0] == case][0]
    plan = plan_for([cam], n_cap=p.shape[1], settings=gs.default_settings(bwd_waves=waves))
    P = _dev(p)
    plan.render(P, n, with_ncontrib=True)
    o = orc.render(p, n, cam)
    Wt = np.random.default_rng(11).uniform(-1, 1, (3, cam["height"], cam["width"])).astype(np.float32)
    Wt[:, o["amb"] != 0] = 0.0
    dL = _dev(Wt).reshape(-1).contiguous()
    r = _store_run(plan)
    gs.gs_raster_bwd_stored(plan.settings, plan.proj_ws, plan.n_cap, plan.n_views, plan.sort_ws, plan.pair_cap,
                            plan.targets_dev, plan.n_targets, plan.total_tiles, r["last"], r["nc"], r["base"],
                            r["store"], dL, plan.accum_ws)
    grad = torch.zeros_like(P)
    gs.gs_project_bwd(plan.settings, P, n, plan.views_dev, plan.n_views, plan.accum_ws, grad)
    ref = orc.render_backward(p, n, cam, Wt)
    ids = np.nonzero(np.linalg.norm(ref[:, :n], axis=0) > 0)[0]
    check_gradients(grad.cpu().numpy().astype(np.float64), ref, ids, f"{case} stored, {waves} waves",
                    p99=0.1 if case == "tiny" else 0.3)
