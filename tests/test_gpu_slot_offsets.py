"""Slot offsets of the per-Gaussian gradients, at the edges of the record
blocks (256) and groups (2048) that they are counted in and past the 2 M
records from which a block takes several groups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views", [(1, 1), (255, 1), (256, 1), (256, 8), (257, 8), (227, 19), (263_000, 8)])
def test_last_views_gradients(n, views):
    """Upstream gradients in the last view only: every other view's slots
    hold zeros, so the sums equal those of the last view planned alone, bit
    for bit.  A later forward of a moved view leaves the slots as they are."""
    import torch
    from paper_2506_02741_amd import render as R
    W, H = (720, 400) if n > 1000 else (64, 48)
    cam = (0.9 * W, 0.9 * W, W / 2, H / 2, W, H)
    rng = np.random.default_rng(n + views)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    k = R.Keyframe(cam, pose, np.sort(rng.choice(W * H, n, replace=False)).astype(np.int32),
                   rng.uniform(1.0, 2.0, n).astype(np.float32), rng.uniform(0, 1, (3, n)).astype(np.float32),
                   rng.uniform(0.05, 0.9, n).astype(np.float32), rng.uniform(0.002, 0.02, n).astype(np.float32),
                   learnable=True).with_grad_buffers()
    poses = []
    for v in range(views):
        p = pose.copy()
        p[:, 3] = rng.uniform(-0.1, 0.1, 3)
        poses.append(p)
    up = torch.as_tensor(rng.normal(size=(3, W * H)).astype(np.float32), device="cuda")

    def grads(run):
        for g in (k.g_color, k.g_opacity, k.g_radius):
            g.zero_()
        run()
        return [g.cpu().numpy().copy() for g in (k.g_color, k.g_opacity, k.g_radius)]
    last = [R.View(cam, p) for p in poses]
    single, _ = R.plan_checked([k], last[-1:], run=lambda p: p.render_fwd())
    ref = grads(lambda: single.render_bwd(up, twist=False))
    plan, _ = R.plan_checked([k], last, run=lambda p: p.render_fwd())
    g = torch.zeros(3, plan.P, device="cuda")
    g[:, plan.offsets[views - 1]:plan.offsets[views - 1] + W * H] = up
    got = grads(lambda: plan.render_bwd(g, twist=False))
    assert np.abs(ref[0]).max() > 0
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    for v in last:
        v.pose[3] += 0.05
    plan.render_fwd()
    for a, b in zip(grads(plan.debug_gather), ref):
        assert np.array_equal(a, b)
