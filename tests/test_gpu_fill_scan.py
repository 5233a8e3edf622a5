"""Plans on both sides of the 512 tiles up to which the key fill sums up the
tile counts itself: lists against the oracle, gradients against a plan of two
views, whose counts are always summed up by the tile scan."""
import numpy as np
import pytest

from test_gpu_parity import np_, same_ranges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(8, 8), (256, 128), (584, 56), (216, 152)])  # 1, 512, 511, 513 tiles of 8
@pytest.mark.parametrize("n,wide", [(40, 0.0), (3000, 0.0), (2500, 0.05)])
def test_lists_and_gradients(orc, W, H, n, wide):
    import torch
    from paper_2506_02741_amd import render as R
    rng = np.random.default_rng(W + n)
    cam = (0.9 * W, 0.9 * W, W / 2, H / 2, W, H)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    n = min(n, W * H)
    pix = np.sort(rng.choice(W * H, n, replace=False)).astype(np.uint32)
    radius = rng.uniform(0.002, 0.02, n) * np.where(rng.random(n) < wide, 40.0, 1.0)
    a = (rng.uniform(1.0, 2.0, n).astype(np.float32), rng.uniform(0, 1, (3, n)).astype(np.float32),
         rng.uniform(0.05, 0.9, n).astype(np.float32), radius.astype(np.float32))
    k = R.Keyframe(cam, pose, pix.astype(np.int32), *a, learnable=True).with_grad_buffers()
    okf = orc.Keyframe(cam, pose, pix, *a)
    prm = R.params(tile=8)
    keys, vals, ranges = orc.tile_lists(orc.ViewSpec(cam, pose), [okf], orc.params(tile=8))
    up = torch.as_tensor(rng.normal(size=(3, W * H)).astype(np.float32), device="cuda")
    grads = []
    for views in (1, 2):
        plan, _ = R.plan_checked([k], [R.View(cam, pose) for _ in range(views)], prm,
                                 run=lambda p: p.render_fwd())
        g = torch.zeros(3, plan.P, device="cuda")
        g[:, :W * H] = up
        for _ in range(2):  # a pass leaves the counters as it found them
            plan.render_fwd()
            st = plan.debug_state()
            assert plan.status() == (0, views * len(vals))
            assert same_ranges(np_(st["ranges"])[:ranges.shape[0]], ranges)
            assert np.array_equal(np_(st["ids"])[:len(vals)].astype(np.uint32), vals)
            for b in (k.g_color, k.g_opacity, k.g_radius):
                b.zero_()
            plan.render_bwd(g, twist=False)
            grads.append([np_(b) for b in (k.g_color, k.g_opacity, k.g_radius)])
    assert np.abs(grads[0][0]).max() > 0
    for other in grads[1:]:
        for x, y in zip(grads[0], other):
            assert np.array_equal(x, y)
