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
