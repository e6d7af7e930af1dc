"""The forward raster's regions and its two waves-per-tile forms against the count variant, which walks every
Gaussian that touches a tile with one pixel a lane: the same images, transmittances and list positions, bit for bit,
on both sides of the tile count that divides the forms, for every tile shape, batch size and schedule."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _params(n, needles, seed=7):
    """n Gaussians; some small, some (needles) long, thin and turned, so that regions are crossed at any angle."""
    p, _, _ = scenes.tiny_scene(seed, n=n)
    rng = np.random.default_rng(seed)
    if needles:
        k = n // 3
        scale = np.log(np.array([[0.8], [0.004], [0.004]])) + 0.5 * rng.standard_normal((3, k))
        p[3:6, :k] = scale
    p[3:6, n // 2:n] -= 1.5
    return torch.as_tensor(np.ascontiguousarray(p, np.float32)).cuda()


@pytest.mark.parametrize("tw", (8, 16, 32))
@pytest.mark.parametrize("w,h", [(17, 9), (150, 110), (640, 900), (802, 963), (1277, 701)])
@pytest.mark.parametrize("needles", (False, True))
def test_forms_agree_with_the_count_variant(tw, w, h, needles):
    from paper_2311_16728_amd.gs import default_settings

    n = 1500
    p = _params(n, needles)
    f = 0.8 * max(w, h)
    cam = scenes.pinhole(w, h, f, f, w / 2 - 3.3, h / 2 + 2.1, R=np.eye(3), t=[0.02, -0.03, 0.1], bg=(0.1, 0.3, 0.2))
    for batch, schedule in ((256, 0), (64, 0), (128, 0), (256, 1)):
        s = default_settings(batch=batch, schedule=schedule)
        plan = plan_for([cam], levels=(0, 1), n_cap=p.shape[1], settings=s, tile_w=tw)
        plan.render(p, n)
        got = [x.clone() for x in (plan.rgb, plan.T, plan.last)]
        assert not plan.overflowed()
        for x in (plan.rgb, plan.T):
            x.fill_(float("nan"))
        plan.last.fill_(-7)
        plan.render_fwd(with_ncontrib=True)
        for a, b in zip(got, (plan.rgb, plan.T, plan.last)):
            assert torch.equal(a, b), (plan.total_tiles, batch, schedule, (a != b).sum().item())
    assert (plan.ncontrib > 0).any()
