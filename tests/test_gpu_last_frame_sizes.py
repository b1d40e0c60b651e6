"""Last-frame search on both sides of its one-workgroup resolve (4096 points) and
at the edges of its waves of 64 points, in every direction of motion, with and
without the rotation check: equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from synth.motion import last_frame_case
from synth.pinhole import pinhole_frame

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_batch_frames=1, max_inflight=1))


@pytest.fixture(scope="module")
def frame():
    return pinhole_frame(91, n_kp=3600, n_map=7000, images=False)


@pytest.mark.parametrize("n,direction,check", [(1, 0, 1), (63, 0, 1), (65, 1, 1), (1153, -1, 1), (1153, 0, 0), (4096, 0, 1),
                                               (4097, 0, 1), (6900, 0, 1), (6900, 1, 0), (6900, -1, 1)])
def test_sizes_and_directions_equal_oracle(ft, ctx, frame, n, direction, check):
    case = last_frame_case(frame, 17, extra_frac=4.0, direction=direction, check_orientation=check)
    case = dict(case, last={k: np.ascontiguousarray(v[:n]) for k, v in case["last"].items()})
    assert len(case["last"]["octave"]) == n
    want = oracle.search_last_frame(case)
    d = ft.DeviceLastFrame(case)
    for _ in range(2):
        d.run(ctx)
    torch.cuda.synchronize()
    got = d.results()
    for k in ("last_match", "last_dist", "kp_match", "n_matches"):
        assert np.array_equal(got[k], want[k]), k
