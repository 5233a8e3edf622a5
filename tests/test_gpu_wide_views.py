"""Gaussians over more than 64 tiles in plans of unequal views: each view's part
of their list goes by its records, and a view with more of them than its part
holds puts the others into the list's rest."""
import numpy as np
import pytest

from test_gpu_parity import np_, same_ranges

pytestmark = pytest.mark.gpu

W, H = 203, 148
CAM = (160.0, 170.0, W / 2, H / 2, W, H)
POSE = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)


def keyframe(orc, n, radii, seed):
    from paper_2506_02741_amd import render as R
    rng = np.random.default_rng(seed)
    pix = rng.integers(0, W * H, n).astype(np.uint32)
    depth = rng.uniform(0.5, 4.0, n).astype(np.float32)
    a = (pix, depth, rng.uniform(0, 1, (3, n)).astype(np.float32),
         rng.uniform(0.05, 0.3, n).astype(np.float32), rng.uniform(*radii, n).astype(np.float32))
    return R.Keyframe(CAM, POSE, pix.astype(np.int32), *a[1:]), orc.Keyframe(CAM, POSE, *a)


@pytest.mark.parametrize("order", [(0, 1), (1, 0), (1, 0, 1, 0)])
def test_lists_of_a_few_wide_records_beside_many_small_ones(orc, order):
    from paper_2506_02741_amd import render as R
    kinds = [keyframe(orc, 300, (0.5, 2.0), 1), keyframe(orc, 100000, (0.002, 0.01), 2)]
    ks, okfs = zip(*[kinds[i] for i in order])
    views = [R.View(CAM, POSE, i, 1) for i in range(len(order))]
    plan = R.Plan(ks, views)
    plan.render_fwd()
    need = plan.status()[1]
    plan = R.Plan(ks, views, pair_capacity=need)
    for _ in range(2):
        plan.render_fwd()
        st = plan.debug_state()
        assert plan.status()[0] == 0
        first, rec, wide = 0, 0, []
        for v, okf in enumerate(okfs):
            _, vals, ranges = orc.tile_lists(orc.ViewSpec(CAM, POSE), [okf], orc.params())
            nt = ranges.shape[0]
            assert same_ranges(np_(st["ranges"])[v * nt:(v + 1) * nt].astype(np.int64) - first, ranges)
            assert np.array_equal(np_(st["ids"])[first:first + len(vals)].astype(np.uint32), vals)
            first += len(vals)
            rc = np_(st["rect"])[rec:rec + ks[v].n]
            rec += ks[v].n
            wide.append(((rc[:, 2] - rc[:, 0] + 1) * (rc[:, 3] - rc[:, 1] + 1) > 64).sum())
        # (the parts are a quarter of the capacity in all)
        v = order.index(0)
        assert wide[v] > need / 4 * ks[v].n / rec + 1 and need == first


@pytest.mark.parametrize("n_views", [2, 49, 130])
def test_wide_records_of_many_views(orc, n_views):
    """Parts of some hundred places each, counted side by side."""
    from paper_2506_02741_amd import render as R
    k, okf = keyframe(orc, 150, (0.5, 2.0), 3)
    poses = np.repeat(POSE[None], n_views, 0)
    poses[:, 2, 3] = np.linspace(0.0, 2.0, n_views)  # from few tiles per record to many
    plan, _ = R.plan_checked([k], [R.View(CAM, p, 0, 1) for p in poses], run=lambda p: p.render_fwd())
    for _ in range(2):
        plan.render_fwd()
        st = plan.debug_state()
        ids, ranges_all, first = np_(st["ids"]).astype(np.uint32), np_(st["ranges"]).astype(np.int64), 0
        for v, p in enumerate(poses):
            _, vals, ranges = orc.tile_lists(orc.ViewSpec(CAM, p), [okf], orc.params())
            nt = ranges.shape[0]
            assert same_ranges(ranges_all[v * nt:(v + 1) * nt] - first, ranges)
            assert np.array_equal(ids[first:first + len(vals)], vals)
            first += len(vals)
        assert plan.status() == (0, first)
