"""Initialiser calls with more work items than one grid dimension holds threads (2^32)."""

import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def test_features_of_more_than_2_to_32_values():
    """26,844,000 keypoints of 160 features: 1,000 keypoints over and over, whose rows have to repeat."""
    from paper_2311_16728_amd import gs

    few, times, H, W = 1000, 26844, 40, 50
    rng = np.random.default_rng(2)
    img = torch.as_tensor(rng.uniform(size=(3, H, W)), dtype=torch.float32).cuda()
    kp = np.stack([rng.uniform(0, W - 1, few), rng.uniform(0, H - 1, few), rng.uniform(1, 5, few), 1.2 ** rng.integers(0, 8, few)], 1)
    kp = torch.as_tensor(kp, dtype=torch.float32).cuda()
    want = torch.full((few, 160), -1, dtype=torch.int16, device="cuda")
    gs.gs_init_features(img, kp, want)
    x = torch.full((few * times, 160), -1, dtype=torch.int16, device="cuda")
    assert x.numel() > 2 ** 32
    gs.gs_init_features(img, kp.repeat(times, 1), x)
    assert (want != -1).all()
    for part in x.view(times, few, 160).split(2000):
        assert torch.equal(part, want.expand_as(part))
