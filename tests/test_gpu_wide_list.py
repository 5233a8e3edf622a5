"""Gaussians over more than 64 tiles: the list they are binned from, past the
256 records of one turn and the 8192 tiles of one round of the tile scan, over
several views, and when the pairs overflow the capacity."""
import numpy as np
import pytest

from test_gpu_parity import np_, same_ranges

pytestmark = pytest.mark.gpu


def scene(orc, n, W, H, n_views, seed):
    from paper_2506_02741_amd import render as R
    cam = (160.0, 170.0, W / 2, H / 2, W, H)
    rng = np.random.default_rng(seed)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    pix = np.sort(rng.choice(W * H, n, replace=False)).astype(np.uint32)
    depth = rng.uniform(0.5, 4.0, n).astype(np.float32)
    radius = np.exp(rng.uniform(np.log(0.05), np.log(2.0), n)).astype(np.float32)
    color = rng.uniform(0, 1, (3, n)).astype(np.float32)
    opacity = rng.uniform(0.05, 0.3, n).astype(np.float32)
    poses = [pose.copy() for _ in range(n_views)]
    for v, p in enumerate(poses):
        p[0, 3] = 0.05 * v
    k = R.Keyframe(cam, pose, pix.astype(np.int32), depth, color, opacity, radius)
    okf = orc.Keyframe(cam, pose, pix, depth, color, opacity, radius)
    return R, cam, poses, k, okf


@pytest.mark.parametrize("n,W,H,views,tile", [(700, 203, 148, 1, 16), (700, 203, 148, 3, 16),
                                              (900, 600, 400, 2, 32), (700, 1000, 600, 1, 8)])
def test_lists_of_wide_gaussians(orc, n, W, H, views, tile):
    """Lists against the oracle, bit for bit, in repeated passes."""
    R, cam, poses, k, okf = scene(orc, n, W, H, views, n + tile)
    plan, _ = R.plan_checked([k], [R.View(cam, p) for p in poses], R.params(tile=tile),
                             run=lambda p: p.render_fwd())
    for _ in range(2):
        plan.render_fwd()
        st = plan.debug_state()
        first, wide = 0, 0
        for v, p in enumerate(poses):
            keys, vals, ranges = orc.tile_lists(orc.ViewSpec(cam, p), [okf], orc.params(tile=tile))
            nt = ranges.shape[0]
            got = np_(st["ranges"])[v * nt:(v + 1) * nt].astype(np.int64) - first
            assert same_ranges(got, ranges)
            assert np.array_equal(np_(st["ids"])[first:first + len(vals)].astype(np.uint32), vals)
            first += len(vals)
            rc = np_(st["rect"])[v * n:(v + 1) * n]
            wide += ((rc[:, 2] - rc[:, 0] + 1) * (rc[:, 3] - rc[:, 1] + 1) > 64).sum()
        assert wide > 256


@pytest.mark.parametrize("cap", [1, 40, 5000])
def test_overflow_by_wide_gaussians(orc, cap):
    """A capacity below the wide records' number, and one between it and the
    pairs: the pass reports what is needed and stays in bounds, and a plan of
    that size renders."""
    from paper_2506_02741_amd import _lib
    R, cam, poses, k, okf = scene(orc, 100, 203, 148, 1, 3)
    views = [R.View(cam, poses[0])]
    plan = R.Plan([k], views, pair_capacity=cap)
    plan.render_fwd()
    rc, need = plan.status()
    keys, vals, ranges = orc.tile_lists(orc.ViewSpec(cam, poses[0]), [okf], orc.params())
    assert rc == _lib.VTGS_E_CAPACITY and need == len(vals)
    plan = R.Plan([k], views, pair_capacity=need)
    plan.render_fwd()
    assert plan.status()[0] == _lib.VTGS_OK
    assert np.array_equal(np_(plan.debug_state()["ids"])[:need].astype(np.uint32), vals)
