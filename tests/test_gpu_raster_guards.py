"""What one Gaussian may reach in the backward raster: a colour that is not finite, or so large that its product with
the loss gradient is not, stays with the pixels that composite it."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, proj_records, require_gpu
from tests.test_gpu_raster_bwd import _accum

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("colour", [float("inf"), 1e38, 1e9])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_colour_stays_with_the_pixels_that_composite_it(colour, waves):
    """One Gaussian's red is infinite, or overflows with the loss gradient (here 100), or is only large.  Gaussians of
    the same tiles that share no pixel with it get what they get beside a plain colour, up to a few float32 roundings
    (the walk with branches adds in another order)."""
    rng = np.random.default_rng(4)
    n, k = 220, 100
    raw = scenes.draw_gaussians(rng, n, (-1, -1, 2.0), (1, 1, 4.0))
    raw[0:3, k], raw[3:6, k], raw[10, k] = (0.1, 0.05, 3.0), np.log(0.05), 0.0
    p = torch.as_tensor(raw).cuda()
    cam = scenes.pinhole(64, 48, 50.0)
    plan = plan_for([cam], n_cap=p.shape[1])
    plan.render(p, n)
    dL = torch.as_tensor(100 * rng.choice([-1, 1], size=3 * 64 * 48), dtype=torch.float32).cuda()
    clean = _accum(plan, dL, waves)[:n]
    # Gaussians with a pixel in common with k: the gradient of the pixels it may reach alone
    mean, cov, _ = (x[k].astype(np.float64) for x in proj_records(plan, n))
    a, b, c = cov[0] + 0.3, cov[1], cov[2] + 0.3
    dx, dy = mean[0] - np.arange(64)[None, :], mean[1] - np.arange(48)[:, None]
    reach = cov[3] * np.exp(-0.5 * (c * dx * dx - 2 * b * dx * dy + a * dy * dy) / (a * c - b * b)) >= 0.999 / 255
    assert 8 < reach.sum() < 200
    touched = (_accum(plan, torch.as_tensor(np.tile(reach, (3, 1, 1)).reshape(-1), dtype=torch.float32).cuda(), waves)[:n]
               != 0).any(dim=1)
    touched[k] = True
    p[11, k] = colour
    plan.render(p, n)
    got = _accum(plan, dL, waves)[:n]
    others = ~touched & (clean != 0).any(dim=1)
    assert int(others.sum()) > n // 3
    assert torch.isfinite(got[others]).all()
    torch.testing.assert_close(got[others], clean[others], rtol=1e-4, atol=1e-5 * float(clean.abs().max()))
    if not np.isfinite(colour):
        assert not torch.isfinite(got[k, :6]).all() and torch.isfinite(got[k, 6:]).all()


@pytest.mark.parametrize("big", [1.0, 1e31])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_gaussian_of_one_tile_repeats_its_bits(waves, big):
    """Gaussians inside a single tile: their sums are the same bits in every run, whatever order its waves finish in
    (big: one pixel's gradient that makes the tile be walked with branches)."""
    rng = np.random.default_rng(6)
    n = 300
    p = torch.as_tensor(scenes.draw_gaussians(rng, n, (-0.2, -0.2, 2.0), (0.2, 0.2, 4.0))).cuda()
    p[3:6] += 1.0
    plan = plan_for([scenes.pinhole(16, 16, 30.0)], n_cap=p.shape[1])
    plan.render(p, n)
    dL = torch.as_tensor(rng.normal(size=3 * 256), dtype=torch.float32).cuda()
    dL[100] *= big
    first = _accum(plan, dL, waves)[:n]
    assert ((first != 0).sum(1) == 9).sum() > n // 2
    for _ in range(40):
        assert torch.equal(_accum(plan, dL, waves)[:n], first)
