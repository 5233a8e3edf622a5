"""Ingestion at the edges of its waves (256 cells) and blocks (1024 cells), on
grids narrower than a wave, and with strides that do not divide the image.
Equal to the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,stride", [(1, 1, 1), (1, 300, 1), (63, 5, 1), (64, 16, 1), (257, 8, 1),
                                        (1023, 1, 1), (205, 5, 1), (33, 200, 3), (130, 71, 7), (5, 5, 9)])
@pytest.mark.parametrize("masked", [False, True])
def test_cells(orc, W, H, stride, masked):
    from paper_2506_02741_amd import render as R
    rng = np.random.default_rng(W * H + stride)
    depth = rng.uniform(0.5, 4.0, (H, W)).astype(np.float32)
    depth[rng.random((H, W)) < 0.2] = 0.0
    depth[rng.random((H, W)) < 0.05] = np.inf
    depth[rng.random((H, W)) < 0.05] = np.nan
    rgb = rng.uniform(0, 1, (3, H, W)).astype(np.float32)
    mask = (rng.random((H, W)) < 0.6).astype(np.uint8) if masked else None
    cam = (50.0, 52.0, W / 2, H / 2, W, H)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    k = R.Keyframe.ingest(depth, rgb, cam, pose, stride, 0.9, mask)
    pix = np.array([y * W + x for y in range(0, H, stride) for x in range(0, W, stride)
                    if np.isfinite(depth[y, x]) and depth[y, x] > 0 and (mask is None or mask[y, x])], np.int64)
    d = depth.ravel()[pix]
    assert k.n == len(pix) and np.array_equal(np_(k.pix), pix)
    assert np.array_equal(np_(k.depth), d)
    assert np.array_equal(np_(k.color), rgb.reshape(3, -1)[:, pix])
    assert np.array_equal(np_(k.opacity), np.full(len(pix), 0.9, np.float32))
    assert np.array_equal(np_(k.radius), np.float32(stride) * d / np.float32(50.0))
