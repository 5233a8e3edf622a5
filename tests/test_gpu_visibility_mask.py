"""The visibility mask without counts (blocks of another size) equals the mask
with counts, which the oracle checks elsewhere, at the edges of its blocks and
over one launch's targets and more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(5, 3), (16, 16), (257, 1), (64, 48), (205, 61)])
@pytest.mark.parametrize("targets", [1, 32, 33])
def test_mask_alone(w, h, targets):
    import torch
    from paper_2506_02741_amd import sections as S
    rng = np.random.default_rng(w * h + targets)
    cam = (0.8 * w, 0.8 * w, w / 2, h / 2, w, h)
    t = lambda x: torch.tensor(np.ascontiguousarray(x, np.float32), device="cuda")
    src = rng.uniform(1.0, 1.03, (h, w))
    src[rng.random((h, w)) < 0.1] = 0.0
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], 1)
    keep = []
    for _ in range(targets):
        p = pose.copy()
        p[:, 3] += rng.uniform(-0.02, 0.02, 3)
        keep.append((t(rng.uniform(1.0, 1.03, h * w)), t(p.reshape(12))))
    refs = [S.frame_ref(d, cam, p) for d, p in keep]
    src, pose = t(src.reshape(-1)), t(pose.reshape(12))
    mask, counts = S.visibility(src, cam, pose, refs)
    alone, none = S.visibility(src, cam, pose, refs, want_counts=False)
    assert none is None and torch.equal(mask, alone)
    if min(w, h) > 2:
        assert 0 < int(mask.sum()) <= int(counts.sum())
