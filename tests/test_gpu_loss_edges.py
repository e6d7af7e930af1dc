"""The loss and the pyramid at sizes around their blocks (32x32 outputs, 30x16), for every tile shape: against the
oracle with the bounds of the parity tests, and what one value that is not finite reaches."""

import numpy as np
import pytest
import torch

import scenes
from tests.gpu_util import plan_for, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _plan(sizes, tw, weights):
    return plan_for([scenes.pinhole(w, h, 50.0) for w, h in sizes], weights=weights, tile_w=tw)


@pytest.mark.parametrize("tw", (8, 16, 32))
@pytest.mark.parametrize("sizes", [[(1, 1)], [(32, 32)], [(33, 31), (5, 70)], [(64, 65), (31, 33), (16, 150)],
                                   [(17, 16)] * 10 + [(130, 43)]])
def test_loss_at_block_edges(orc, sizes, tw):
    weights = [1.0 + 0.25 * i for i in range(len(sizes))]
    plan = _plan(sizes, tw, weights)
    rng = np.random.default_rng(11)
    xs = [rng.uniform(size=(3, h, w)).astype(np.float32) for w, h in sizes]
    ys = [rng.uniform(size=(3, h, w)).astype(np.float32) for w, h in sizes]
    x = np.concatenate([a.reshape(-1) for a in xs])
    y = np.concatenate([a.reshape(-1) for a in ys])
    plan.rgb.copy_(torch.as_tensor(x))
    plan.loss_ws.fill_(255)   # (nothing may be read that was not written)
    plan.dL.fill_(float("nan"))
    plan.loss(torch.as_tensor(y).cuda(), 0.2, True)
    got, total = plan.dL.cpu().numpy(), 0.0
    for i, (w, h) in enumerate(sizes):
        L, d, _ = orc.loss(xs[i], ys[i], 0.2)
        off = plan.target_slice(i)[0]
        g = got[3 * off:3 * (off + w * h)].reshape(3, h, w)
        total += weights[i] * L
        assert float(plan.d_loss[i]) == pytest.approx(L, rel=2e-5)
        assert np.abs(g - weights[i] * d).max() <= 2e-4 * np.abs(weights[i] * d).max()
    assert float(plan.d_total[0]) == pytest.approx(total, rel=2e-5)


@pytest.mark.parametrize("value", (float("nan"), float("inf")))
def test_what_is_not_finite_stays_in_its_windows(value):
    w, h, px, py = 97, 75, 40, 33
    plan = _plan([(w, h)], 16, [1.0])
    rng = np.random.default_rng(5)
    x = rng.uniform(size=(3, h, w)).astype(np.float32)
    y = torch.as_tensor(rng.uniform(size=3 * h * w).astype(np.float32)).cuda()
    grads = []
    for v in (x[1, py, px], value):
        x[1, py, px] = v
        plan.rgb.copy_(torch.as_tensor(x.reshape(-1)))
        plan.loss(y, 0.2, True)
        grads.append(plan.dL.cpu().numpy().reshape(3, h, w).copy())
    reach = np.zeros((3, h, w), bool)
    reach[1, py - 10:py + 11, px - 10:px + 11] = True
    assert np.array_equal(grads[0][~reach], grads[1][~reach])
    assert not np.isfinite(grads[1][1, py, px])
    assert not np.isfinite(float(plan.d_total[0]))


@pytest.mark.parametrize("C,H,W,levels", [(3, 1, 1, 2), (1, 2, 3, 16), (3, 31, 59, 3), (3, 32, 60, 2), (3, 33, 61, 4),
                                          (2, 65, 121, 3), (70000, 2, 3, 2), (3, 40, 40, 1)])
def test_pyramid_at_block_edges(orc, C, H, W, levels):
    from paper_2311_16728_amd import gs

    img = np.random.default_rng(9).uniform(size=(C, H, W)).astype(np.float32)
    want = orc.pyramid(img, levels)
    out = torch.full((sum(a.size for a in want) + 64,), float("nan"), device="cuda")
    gs.gs_pyramid_build(torch.as_tensor(img).cuda(), levels, out)
    o, at = out.cpu().numpy(), 0
    for lv in want:
        assert np.abs(o[at:at + lv.size].reshape(lv.shape) - lv).max() <= 1e-6
        at += lv.size
    assert np.isnan(o[at:]).all()
    assert np.array_equal(o[:img.size].reshape(img.shape), img)
