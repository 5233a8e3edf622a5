"""The tile sort where depths are equal or a few steps of a float apart (its
buckets then go by depth and id) and long lists in plans of mostly short ones
(sorted as runs by the short lists' kernel): against the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import np_, same_ranges
from test_gpu_tile_sort import R, depths  # noqa: F401 (R: a fixture)

pytestmark = pytest.mark.gpu
POSE = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)


def check_lists(R, orc, kcam, cam, pix, depth, rng):
    n = len(pix)
    color, opacity = rng.uniform(0, 1, (3, n)).astype(np.float32), np.full(n, 0.5, np.float32)
    radius = np.full(n, 0.01, np.float32)
    plan = R.Plan([R.Keyframe(kcam, POSE, pix.astype(np.int32), depth, color, opacity, radius)], [R.View(cam, POSE)])
    plan.render_fwd()
    st = plan.debug_state()
    assert plan.status()[0] == 0
    okf = orc.Keyframe(kcam, POSE, pix.astype(np.uint32), depth, color, opacity, radius)
    _, vals, ranges = orc.tile_lists(orc.ViewSpec(cam, POSE), [okf])
    assert same_ranges(np_(st["ranges"]), ranges)
    assert np.array_equal(np_(st["ids"])[:len(vals)].astype(np.uint32), vals)
    return ranges


# steps from the nearest depth of the list to each Gaussian's
STEPS = {"one": lambda n, rng: np.zeros(n, np.int64),
         "neighbours": lambda n, rng: rng.integers(0, 4, n),
         "levels": lambda n, rng: 4194 * rng.integers(0, 3, n) + rng.integers(0, 2, n),
         "below": lambda n, rng: np.append(rng.integers(0, 65536, n - 1), 65535),
         "above": lambda n, rng: np.append(rng.integers(0, 65537, n - 1), 65536)}


@pytest.mark.parametrize("spread", [False, True])
@pytest.mark.parametrize("kind", sorted(STEPS))
@pytest.mark.parametrize("n", [2, 700, 3000, 8193])
def test_near_depths(R, orc, n, kind, spread):  # noqa: F811
    rng = np.random.default_rng(n)
    kcam, cam = (20.0, 20.0, 8.0, 8.0, 1024, 16), (20.0, 20.0, 8.0, 8.0, 16, 16)
    steps = STEPS[kind](n, rng)
    steps[0] = 0
    near = (np.float32(2.0).view(np.uint32) + steps.astype(np.uint32)).view(np.float32)
    # spread: the tile's ids lie anywhere among 150,000 Gaussians, the others
    # outside the view
    total = 150000 if spread else n
    ids = np.sort(rng.choice(total, n, replace=False))
    pix, depth = np.full(total, 8 * 1024 + 1000), np.full(total, 2.0, np.float32)
    pix[ids] = 8 * 1024 + 8
    depth[ids] = near
    ranges = check_lists(R, orc, kcam, cam, pix, depth, rng)
    assert np.asarray(ranges).reshape(-1).max() == n


@pytest.mark.parametrize("kind", ["uniform", "outliers", "quantised", "equal"])
@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049, 3073])
def test_long_lists_among_short_ones(R, orc, n, kind):  # noqa: F811
    rng = np.random.default_rng(n)
    cam = (20.0, 20.0, 168.0, 120.0, 320, 240)
    check_lists(R, orc, cam, cam, np.full(n, 120 * 320 + 168), depths(kind, n, rng).astype(np.float32), rng)
