"""Binning of Gaussians whose tile rectangles are too wide for a shared box:
small ones counted in the wave's own counters, those of more than 64 tiles from a
list.  Lists against the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import check_images, np_, oracle_ref, same_ranges

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    torch.cuda.set_device(0)
    from paper_2506_02741_amd import render
    return render


@pytest.mark.parametrize("n,views", [(1, 1), (64, 1), (333, 1), (100, 2)])
@pytest.mark.parametrize("tile", [8, 16])
def test_wide_rectangles(R, orc, n, views, tile):
    """Radii from a pixel to several images' width (rectangles of 1, around
    64, and all tiles), records of two views in one wave where there are two
    views."""
    W, H = 203, 148
    cam = (160.0, 170.0, W / 2, H / 2, W, H)
    rng = np.random.default_rng(n * 10 + tile)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    pix = np.sort(rng.choice(W * H, n, replace=False)).astype(np.uint32)
    depth = rng.uniform(0.5, 4.0, n).astype(np.float32)
    radius = np.exp(rng.uniform(np.log(0.003), np.log(2.0), n)).astype(np.float32)
    color = rng.uniform(0, 1, (3, n)).astype(np.float32)
    opacity = rng.uniform(0.05, 0.3, n).astype(np.float32)
    moved = pose.copy()
    moved[0, 3] = 0.05
    poses = [pose, moved][:views]
    k = R.Keyframe(cam, pose, pix.astype(np.int32), depth, color, opacity, radius)
    prm = R.params(tile=tile)
    plan, imgs = R.plan_checked([k], [R.View(cam, p) for p in poses], prm, pair_capacity=n * views * 600,
                                run=lambda p: p.render_fwd())
    st = plan.debug_state()
    okf = orc.Keyframe(cam, pose, pix, depth, color, opacity, radius)
    first, areas = 0, []
    for v, p in enumerate(poses):
        ov = orc.ViewSpec(cam, p)
        keys, vals, ranges = orc.tile_lists(ov, [okf], orc.params(tile=tile))
        nt = ranges.shape[0]
        got = np_(st["ranges"])[v * nt:(v + 1) * nt].astype(np.int64) - first
        assert same_ranges(got, ranges)
        assert np.array_equal(np_(st["ids"])[first:first + len(vals)].astype(np.uint32), vals)
        first += len(vals)
        P = W * H
        check_images(*[x[..., v * P:(v + 1) * P] for x in imgs], oracle_ref(orc, ov, [okf]))
        rc = np_(st["rect"])[v * n:(v + 1) * n]
        areas.append((rc[:, 2] - rc[:, 0] + 1) * (rc[:, 3] - rc[:, 1] + 1))
    if n > 64:
        a = np.concatenate(areas)
        assert (a > 64).any() and ((a > 24) & (a <= 64)).any()
