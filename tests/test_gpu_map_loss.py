"""Eq. 2 and its image gradients at the edges of the SSIM kernels' blocks (16 x
16 and 32 x 16 pixels, windows of 11), of the L1 blocks (256 pixels) and with
views of different sizes in one plan."""
import numpy as np
import pytest

from test_gpu_parity import grad_close, np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[(1, 1)], [(31, 15)], [(32, 16), (33, 17)], [(65, 40), (5, 70), (16, 16)],
                                   [(257, 1), (64, 49)]])
@pytest.mark.parametrize("learnable", [True, False])
def test_map_loss_at_block_edges(orc, sizes, learnable):
    """On the GPU's own images the loss within 1e-5 and the gradients within
    1e-3 of the FP64 oracle's (FP64 evaluation, rounded to FP32 once)."""
    import torch
    from paper_2506_02741_amd import render as R
    rng = np.random.default_rng(len(sizes) + sizes[0][0])
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    W0, H0 = sizes[0]
    n = min(W0 * H0, 300)
    k = R.Keyframe((60.0, 60.0, W0 / 2, H0 / 2, W0, H0), pose,
                   np.sort(rng.choice(W0 * H0, n, replace=False)).astype(np.int32),
                   rng.uniform(1.0, 2.0, n).astype(np.float32), rng.uniform(0, 1, (3, n)).astype(np.float32),
                   rng.uniform(0.3, 0.9, n).astype(np.float32), rng.uniform(0.01, 0.05, n).astype(np.float32),
                   learnable=learnable)
    if learnable:
        k.with_grad_buffers().with_adam()
    views, obs = [], []
    for W, H in sizes:
        rgb = rng.uniform(0, 1, (3, H, W)).astype(np.float32)
        dep = (rng.uniform(1, 2, (H, W)) * (rng.random((H, W)) < 0.8)).astype(np.float32)
        obs.append((rgb, dep))
        views.append(R.View((60.0, 60.0, W / 2, H / 2, W, H), pose, 0, 1, rgb, dep))
    plan = R.Plan([k], views)
    step = torch.zeros(1, dtype=torch.int32, device="cuda")
    for t in (1, 2):
        loss = np_(plan.map_step(step, R.map_cfg(rho=0.8, tau=0.2, sigma=1.0)))
        assert plan.status()[0] == 0 and int(step.item()) == t
        img, gimg = (np_(x).astype(np.float64) for x in plan.debug_images())
        for v, ((W, H), (rgb, dep)) in enumerate(zip(sizes, obs)):
            sl = slice(plan.offsets[v], plan.offsets[v] + W * H)
            L, g_rgb, g_d = orc.map_loss(H, W, img[:3, sl], img[3, sl], rgb, dep, 0.8, 0.2, 1.0)
            assert abs(loss[v] - L) <= 1e-5 * abs(L), (t, v, loss[v], L)
            for got, ref in ((gimg[:3, sl], g_rgb), (gimg[3, sl], g_d)):
                ok, worst = grad_close(got, ref, "view %d" % v)
                assert ok, worst
