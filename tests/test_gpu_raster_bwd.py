"""The backward raster's wave sums and branch-free walk where they can go wrong: every number of staged Gaussians
around its group and stage sizes, every tile shape and wave count, and loss gradients that are not finite."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _accum(plan, dL, waves):
    from paper_2311_16728_amd import gs

    s = type(plan.settings).from_buffer_copy(plan.settings)
    s.bwd_waves = waves
    gs.gs_raster_bwd(s, plan.proj_ws, plan.n_cap, plan.n_views, plan.sort_ws, plan.pair_cap, plan.targets_dev,
                     plan.n_targets, plan.total_tiles, plan.T, plan.last, dL, plan.accum_ws)
    return plan.accum_ws[:36 * plan.n_cap * plan.n_views].view(torch.float32).reshape(-1, 9).double().cpu()


def _reference(p, n, cam, dL):
    """Colour and opacity gradients of the compositing (Eq. 3) by float64 autograd over dense pixels, from the
    projection records' values."""
    from tests.gpu_util import proj_records

    plan = plan_for([cam], n_cap=p.shape[1])
    plan.render(p, n)
    mean, cov, rgbz = (torch.as_tensor(x[:n], dtype=torch.float64) for x in proj_records(plan, n))
    order = torch.argsort(rgbz[:, 3], stable=True)
    order = order[cov[order, 3] >= 1.0 / 255.0]
    W, H = cam["width"], cam["height"]
    yy, xx = torch.meshgrid(torch.arange(H, dtype=torch.float64), torch.arange(W, dtype=torch.float64), indexing="ij")
    leaf = torch.cat([mean, cov, rgbz[:, :3]], 1)[order].requires_grad_(True)
    mx, my, a, b, c, o = (leaf[:, i] for i in range(6))
    a, c = a + 0.3, c + 0.3
    det = a * c - b * b
    dx, dy = mx - xx.reshape(-1, 1), my - yy.reshape(-1, 1)
    at = o * torch.exp(-0.5 * (c * dx * dx - 2 * b * dx * dy + a * dy * dy) / det)
    with torch.no_grad():
        alpha = torch.where(at >= 1.0 / 255.0, at.clamp_max(0.99), 0.0)
        keep = (alpha > 0) & (torch.cumprod(1 - alpha, 1) >= 1e-4)
    alpha = torch.where(keep, at.clamp_max(0.99), 0.0)
    before = torch.cumprod(torch.cat([torch.ones_like(alpha[:, :1]), 1 - alpha[:, :-1]], 1), 1)
    img = ((alpha * before) @ leaf[:, 6:9]).T.reshape(3, H, W)
    (img * dL.double().cpu().reshape(3, H, W)).sum().backward()
    grad = torch.zeros(n, 9, dtype=torch.float64)
    grad[order] = leaf.grad
    grad[:, 3] *= 0.5   # the off-diagonal covariance entry stands for both of the matrix
    return grad


@pytest.mark.parametrize("n", [1, 5, 6, 7, 63, 64, 65, 255, 256, 257, 300])
def test_sums_over_group_and_stage_edges(n):
    """n Gaussians over a ragged 37x29 image, one, two and four waves, against float64.  Bound: float32 sums of a few
    hundred terms of either sign, 2e-4 of the norm per quantity (a flipped cutoff decision of one pixel of the
    thousand is 1/255 of one term)."""
    rng = np.random.default_rng(n)
    p = scenes.draw_gaussians(rng, n, (-0.5, -0.4, 2.0), (0.5, 0.4, 4.0))
    p[3:6, :n] += 0.7
    p = torch.as_tensor(p).cuda()
    cam = scenes.pinhole(37, 29, 60.0)
    dL = torch.as_tensor(rng.normal(size=3 * 37 * 29), dtype=torch.float32).cuda()
    want = _reference(p, n, cam, dL)
    scale = want.norm(dim=0).clamp_min(1e-12)
    for tile_w in (8, 16, 32):
        plan = plan_for([cam], n_cap=p.shape[1], tile_w=tile_w)
        plan.render(p, n)
        for waves in (1, 2, 4):
            got = _accum(plan, dL, waves)[:n]
            err = ((got - want).norm(dim=0) / scale).max().item()
            assert err <= 2e-4, (tile_w, waves, err)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 3e38])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_non_finite_pixel_stays_with_its_gaussians(bad, waves):
    """One pixel's loss gradient is not finite (or near overflow): the Gaussians it composites get non-finite sums
    (finite ones near overflow), every other Gaussian exactly what it gets without that pixel's tile changing."""
    rng = np.random.default_rng(3)
    n = 200
    p = scenes.draw_gaussians(rng, n, (-1, -1, 2.0), (1, 1, 4.0))
    p = torch.as_tensor(p).cuda()
    cam = scenes.pinhole(64, 48, 50.0)
    plan = plan_for([cam], n_cap=p.shape[1])
    plan.render(p, n)
    dL = torch.as_tensor(rng.normal(size=3 * 64 * 48), dtype=torch.float32).cuda()
    clean = _accum(plan, dL, waves)[:n]
    # the Gaussians that the pixel composites: a gradient of one at it alone
    one = torch.zeros_like(dL)
    one[20 * 64 + 33] = 1.0
    touched = (_accum(plan, one, waves)[:n] != 0).any(dim=1)
    assert 0 < int(touched.sum()) < n // 2
    worse = dL.clone()
    worse[20 * 64 + 33] = bad
    got = _accum(plan, worse, waves)[:n]
    if np.isfinite(bad):
        assert (got[touched][:, 6].abs() > 1e30).any()
    else:
        assert (~torch.isfinite(got[touched])).any(dim=1).all()
    assert torch.isfinite(got[~touched]).all()
    # the careful walk adds in another order: a few float32 roundings of sums whose terms are of order one
    torch.testing.assert_close(got[~touched], clean[~touched], rtol=1e-4, atol=1e-4 * float(clean.abs().max()))
