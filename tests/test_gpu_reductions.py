"""Block-wise reductions behind the visibility counts and the keyframe pose
gradients, at the edges of their blocks, launches and target batches."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,n_targets", [(33, 1, 1), (64, 16, 31), (41, 25, 32), (93, 11, 33), (70, 30, 65)])
def test_visibility_counts_over_blocks_and_launches(orc, w, h, n_targets):
    """Pixel counts around the 1024-pixel block and target counts around the
    32 of one launch: masks and counts are integers, equal to the oracle's."""
    import torch
    from paper_2506_02741_amd import sections as S
    rng = np.random.default_rng(w * 100 + n_targets)
    cam = (40.0, 42.0, w / 2, h / 2, w, h)

    def depth():
        return (2.0 + 0.01 * rng.normal(size=(h, w)) * (rng.random((h, w)) < 0.5)
                ).astype(np.float32) * (rng.random((h, w)) < 0.9)

    def pose():
        T = np.eye(4, dtype=np.float32)[:3].copy()
        T[:, 3] = rng.uniform(-0.02, 0.02, 3)
        return T
    src, sp = depth(), pose()
    tgts = [(depth(), cam, pose()) for _ in range(n_targets)]
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a).ravel(), device="cuda")
    keep = [(dev(d), dev(p)) for d, _, p in tgts]
    mask, counts = S.visibility(dev(src), cam, dev(sp), [S.frame_ref(d, cam, p) for d, p in keep])
    vis, cref = orc.visibility(src, cam, sp, tgts)
    assert np.array_equal(counts.cpu().numpy().astype(np.int64), cref)
    assert np.array_equal(mask.cpu().numpy().astype(bool), vis.any(0))
