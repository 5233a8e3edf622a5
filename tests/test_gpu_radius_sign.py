"""Gradients at negative radii.  A Gaussian's image depends on r^2 alone, so
images and the gradients to everything else are those of |r|, and dL/dr
changes its sign with r: bit for bit, and against the oracle."""
import numpy as np
import pytest

from test_gpu_parity import MARGIN, grad_close, np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("geo", [False, True])
@pytest.mark.parametrize("twist", [False, True])
def test_gradients_at_negative_radii(orc, twist, geo):
    import torch
    from paper_2506_02741_amd import render as R
    W, H, n = 80, 60, 700
    cam = (75.0, 78.0, 40.0, 30.0, W, H)
    rng = np.random.default_rng(7)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    vpose = pose.copy()
    vpose[:, 3] = (0.03, -0.02, 0.05)
    attr = [(np.sort(rng.choice(W * H, n, replace=False)).astype(np.uint32),
             rng.uniform(1.0, 2.0, n).astype(np.float32), rng.uniform(0, 1, (3, n)).astype(np.float32),
             rng.uniform(0.05, 0.9, n).astype(np.float32), rng.uniform(0.01, 0.05, n).astype(np.float32))
            for _ in range(2)]
    sign = np.where(rng.uniform(size=n) < 0.5, -1.0, 1.0).astype(np.float32)
    okfs = [orc.Keyframe(cam, pose, p, d, c, o, r * sign) for p, d, c, o, r in attr]
    ov = orc.ViewSpec(cam, vpose, 0, 2)
    up = rng.normal(size=(3, W * H)).astype(np.float32)
    up[:, orc.render(ov, okfs, margin=MARGIN)["marginal"]] = 0.0

    def run(s):
        # the second keyframe is frozen: its records lie between the others
        ks = [R.Keyframe(cam, pose, p.astype(np.int32), d, c, o, r * s, learnable=i == 0)
              for i, (p, d, c, o, r) in enumerate(attr)]
        ks[0].with_grad_buffers()
        if geo:
            ks[0].with_geometry_grads()
        plan, out = R.plan_checked(ks, [R.View(cam, vpose, 0, 2)], run=lambda p: p.render_fwd())
        tw = plan.render_bwd(torch.as_tensor(up, device="cuda"), twist=twist)
        k = ks[0]
        rest = list(out) + [k.g_color, k.g_opacity] + ([tw] if twist else []) + \
            ([k.g_depth, k.g_pose] if geo else [])
        return [np_(t).copy() for t in rest], np_(k.g_radius).copy()

    rest_p, gr_p = run(np.float32(1.0))
    rest_s, gr_s = run(sign)
    assert np.abs(gr_p).max() > 0
    for a, b in zip(rest_p, rest_s):
        assert np.array_equal(a, b)
    assert np.array_equal(gr_s, gr_p * sign)
    gref = orc.render_bwd(ov, okfs, up)
    ok, worst = grad_close(gr_s, gref["radius"][:n], "radius", gref["mag"]["radius"][:n])
    assert ok, worst
