"""Records of keyframes that share blocks of 256 records with others or fill
them alone, and of image widths and pixel indexes on both sides of the
preprocess's short division.  Bit for bit against the oracle."""
import numpy as np
import pytest

from test_gpu_parity import np_, same_ranges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kfs", [[(7, 40, 200)], [(8, 40, 256)], [(9, 40, 257), (8, 9, 3)], [(640, 480, 1000)],
                                 [(5000, 4000, 700)], [(64, 48, 1), (64, 48, 255), (33, 20, 512), (64, 48, 5)],
                                 [(64, 48, 300)] * 7])
@pytest.mark.parametrize("views", [1, 3])
def test_records_bitwise(orc, kfs, views):
    from paper_2506_02741_amd import render as R
    rng = np.random.default_rng(sum(n for _, _, n in kfs) + views)
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)

    def moved(s):
        a = rng.uniform(-0.05, 0.05)
        p = pose.copy()
        p[:2, :2] = [[np.cos(a), -np.sin(a)], [np.sin(a), np.cos(a)]]
        p[:, 3] = rng.uniform(-s, s, 3)
        return p
    ks, okfs = [], []
    for W, H, n in kfs:
        cam = (1.0 * max(W, H), 1.1 * max(W, H), W / 2, H / 2, W, H)
        pix = np.sort(rng.choice(W * H, n, replace=False)).astype(np.uint32)
        pix[-1] = W * H - 1
        a = (rng.uniform(0.8, 3.0, n).astype(np.float32), rng.uniform(0, 1, (3, n)).astype(np.float32),
             rng.uniform(0.05, 0.9, n).astype(np.float32), rng.uniform(0.005, 0.1, n).astype(np.float32))
        kp = moved(0.05)
        ks.append(R.Keyframe(cam, kp, pix.astype(np.int32), *a))
        okfs.append(orc.Keyframe(cam, kp, pix, *a))
    vcam = (70.0, 72.0, 40.0, 30.0, 80, 60)
    poses = [moved(0.1) for _ in range(views)]
    plan, _ = R.plan_checked(ks, [R.View(vcam, p, 0, len(ks)) for p in poses], run=lambda p: p.render_fwd())
    st = plan.debug_state()
    N, first = sum(n for _, _, n in kfs), 0
    for v, p in enumerate(poses):
        ov = orc.ViewSpec(vcam, p, 0, len(ks))
        rec = orc.preprocess32(ov, okfs, orc.params())
        g, rect = np_(st["records"])[v * N:(v + 1) * N], np_(st["rect"])[v * N:(v + 1) * N]
        valid = rec["count"] > 0
        assert valid.any() and np.array_equal(rect[:, 0] <= rect[:, 2], valid)
        assert np.array_equal(rect[valid], rec["rect"][valid])
        for col, name in ((0, "mx"), (1, "my"), (2, "qa"), (3, "qb"), (4, "qc"), (6, "pz"), (7, "ext")):
            assert np.array_equal(g[valid, col], rec[name][valid]), name
        keys, vals, ranges = orc.tile_lists(ov, okfs, orc.params())
        nt = ranges.shape[0]
        got = np_(st["ranges"])[v * nt:(v + 1) * nt].astype(np.int64) - first
        assert same_ranges(got, ranges)
        assert np.array_equal(np_(st["ids"])[first:first + len(vals)].astype(np.uint32), vals)
        first += len(vals)
