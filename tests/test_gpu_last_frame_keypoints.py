"""Last-frame search on both sides of the keypoint count (8192) up to which one
workgroup resolves it: equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from synth.motion import last_frame_case
from synth.pinhole import pinhole_frame

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction,check", [(0, 1), (1, 1), (-1, 0)])
@pytest.mark.parametrize("n_kp", [8192, 8193, 16385])
def test_keypoint_counts_equal_oracle(ft, n_kp, direction, check):
    ctx = ft.Context(ft.default_limits(max_kp_per_image=16400, max_batch_frames=1, max_inflight=1))
    frame = pinhole_frame(92, n_kp=n_kp, n_map=1500, images=False)
    case = last_frame_case(frame, 18, direction=direction, check_orientation=check)
    assert case["kps"]["x"].size == n_kp
    want = oracle.search_last_frame(case)
    assert want["n_matches"] > 100
    d = ft.DeviceLastFrame(case)
    for _ in range(2):
        d.run(ctx)
    torch.cuda.synchronize()
    got = d.results()
    for k in ("last_match", "last_dist", "kp_match", "n_matches"):
        assert np.array_equal(got[k], want[k]), k
