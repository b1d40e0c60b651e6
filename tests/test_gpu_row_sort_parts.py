"""Batches of pinhole frames whose row sorts (eight level bins) run in four parts
(64 sorts or fewer in the launch), two (128 or fewer) and one: equal to the
oracle.  A frame with one view has two sorts."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import bit_equal, compare_frame

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 32, 33, 64, 65, 80])
def test_parts_equal_oracle(ft, n):
    ctx = ft.Context(ft.default_limits(max_kp_per_image=1024, max_map_points=512, max_batch_frames=n, max_inflight=1))
    base = [synth.tiny_pinhole(300 + s, n_kp=40 + 210 * s, n_map=100 + 90 * s) for s in range(4)]
    for f in base:
        assert 8 * f["stereo_cam"]["rows"] <= 8192          # a bin per level and row
        f["right"]["octave"][:] = np.sort(f["right"]["octave"])[::-1] if f is base[2] else f["right"]["octave"]
    want = [oracle.run_frame(f) for f in base]
    frames = [ft.DeviceFrame(base[(3 * i) % 4], "cuda") for i in range(n)]
    for _ in range(2):
        ctx.ft_batch_wait(ctx.ft_batch_submit([f.job() for f in frames]))
    torch.cuda.synchronize()
    got = [f.results() for f in frames]
    for i in range(min(n, 4)):
        compare_frame(got[i], want[(3 * i) % 4])
    for i in range(4, n):
        bit_equal(got[i], got[i % 4])
