"""The tile sort at the edges of its block sizes and at the depth
distributions its buckets meet: one tile that holds every Gaussian, lists
against the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import np_, same_ranges

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    torch.cuda.set_device(0)
    from paper_2506_02741_amd import render
    return render


def depths(kind, n, rng):
    if kind == "uniform":
        return rng.uniform(1.0, 3.0, n)
    if kind == "outliers":     # a surface of a few millimetres, some far ones
        d = 2.0 + 0.003 * rng.uniform(size=n)
        d[rng.uniform(size=n) < 0.02] = rng.uniform(0.02, 500.0)
        return d
    if kind == "quantised":    # runs of equal depth, longer than a bucket takes
        return np.round(rng.uniform(1.0, 1.02, n), 3)
    return np.full(n, 1.5)     # "equal": the order is the id order alone


@pytest.mark.parametrize("kind", ["uniform", "outliers", "quantised", "equal"])
@pytest.mark.parametrize("n", [2, 255, 1024, 1025, 4096, 4097, 8192, 8193, 20000])
def test_list_sizes_and_depth_distributions(R, orc, n, kind):
    rng = np.random.default_rng(n)
    W = H = 16
    cam = (20.0, 20.0, 8.0, 8.0, W, H)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    pix = np.full(n, 8 * W + 8, np.uint32)
    depth = depths(kind, n, rng).astype(np.float32)
    color = rng.uniform(0, 1, (3, n)).astype(np.float32)
    opacity = np.full(n, 0.5, np.float32)
    radius = np.full(n, 0.01, np.float32)
    k = R.Keyframe(cam, pose, pix.astype(np.int32), depth, color, opacity, radius)
    plan = R.Plan([k], [R.View(cam, pose)])
    plan.render_fwd()
    st = plan.debug_state()
    assert plan.status()[0] == 0
    okf = orc.Keyframe(cam, pose, pix, depth, color, opacity, radius)
    keys, vals, ranges = orc.tile_lists(orc.ViewSpec(cam, pose), [okf])
    assert len(vals) == n
    assert same_ranges(np_(st["ranges"]), ranges)
    assert np.array_equal(np_(st["ids"])[:n].astype(np.uint32), vals)
