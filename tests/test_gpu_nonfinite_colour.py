"""Gaussians of non-finite colour: a pixel outside q_cut keeps its value, also
where the coverage bound lets the entry through and the exact test refuses it."""
import numpy as np
import pytest

from test_gpu_parity import np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,batch", [(8, 128), (16, 256), (16, 128), (32, 256)])
def test_pixels_outside_the_cut_stay_finite(tile, batch):
    from paper_2506_02741_amd import render as R
    W, H, n = 480, 440, 48
    cam = (400.0, 410.0, 240.0, 220.0, W, H)
    rng = np.random.default_rng(tile + batch)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    # a wide Gaussian per view, whose cut runs through some thousand pixels
    pix = rng.integers(100, 300, n) * W + rng.integers(100, 380, n)
    rad = rng.uniform(0.05, 0.15, n)

    def run(c):
        ks = [R.Keyframe(cam, pose, pix[i:i + 1].astype(np.int32), np.ones(1, np.float32),
                         np.array([[c], [c], [0.5]], np.float32), np.full(1, 0.9, np.float32),
                         rad[i:i + 1].astype(np.float32)) for i in range(n)]
        # (alpha_min 0: a pixel has coverage exactly where q <= q_cut)
        _, out = R.plan_checked(ks, [R.View(cam, pose, i, 1) for i in range(n)],
                                R.params(tile=tile, batch=batch, alpha_min=0.0), run=lambda p: p.render_fwd())
        return [np_(t).copy() for t in out]
    rgb, depth, sil = run(0.25)
    outside = sil == 0
    assert outside.any() and not outside.all() and np.all(rgb[:, outside] == 0)
    for c in (np.inf, -np.inf, np.nan):
        got, d, s = run(c)
        assert np.array_equal(d, depth) and np.array_equal(s, sil) and np.array_equal(got[2], rgb[2])
        assert np.all(got[:, outside] == 0), int((got[0, outside] != 0).sum())
        assert not np.isfinite(got[:2, ~outside]).any()
