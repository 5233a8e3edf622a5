"""Ingestion on a stream of the caller's that is still busy: its count is read
when that stream has written it."""
import numpy as np
import pytest

from scenes import room_frames
from test_gpu_parity import np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("colours", [True, False])
def test_ingest_on_a_busy_stream(colours):
    import torch
    from paper_2506_02741_amd import render as R
    cam, frames, _ = room_frames(4, 160, 120)
    f = frames[0]
    mask = (np.random.default_rng(1).uniform(size=f.depth.shape) < 0.5).astype(np.uint8)
    args = (f.depth, f.rgb if colours else None, cam.as_tuple(), f.pose, 1, 0.9, mask)
    ref = R.Keyframe.ingest(*args)
    side = torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)
        k = R.Keyframe.ingest(*args, stream=side)
        assert k.n == ref.n
        for a in ("pix", "depth", "color", "opacity", "radius"):
            assert np.array_equal(np_(getattr(k, a)), np_(getattr(ref, a))), a
