"""Pinhole refinement at the edges of its row loads: windows in the four corners
of every pyramid level (the first and last bytes of the pyramid among them), every
alignment of the pyramid in memory, and images of 0 and 255 alone, whose sums are
the largest: equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import compare_frame

pytestmark = pytest.mark.gpu


def corner_frame(seed, shift, noise):
    """A frame whose first keypoints lie in the corners of each level's reach, in
    pairs of one descriptor; pyramids that begin `shift` bytes into their memory."""
    f = synth.tiny_pinhole(seed, n_kp=300, n_map=40)
    f["map"] = {k: v[:0] for k, v in f["map"].items()}
    r = np.random.default_rng(seed)
    for side in ("left", "right"):
        p = dict(f["pyr_" + side])
        data = np.asarray(p["data"])
        if noise:
            data = np.where(r.random(data.size) < 0.5, 0, 255).astype(data.dtype)
        p["data"] = np.concatenate([np.zeros(shift, data.dtype), data])
        p["offset"] = [int(o) + shift for o in p["offset"]]
        f["pyr_" + side] = p
    sf = np.asarray(f["scales"]["sf"], np.float32)
    k = 0
    for lv, (w, h) in enumerate(zip(f["pyr_left"]["width"], f["pyr_left"]["height"])):
        for y in (5, h - 6):
            for xl, xr in ((15, 10), (w - 6, w - 11), (16, 11), (w - 7, w - 12), (5, 10)):
                for side, x in (("left", xl), ("right", xr)):
                    d = f[side]
                    d["x"][k], d["y"][k], d["octave"][k] = x * sf[lv], y * sf[lv], lv
                f["left"]["desc"][k] = f["right"]["desc"][k] = r.integers(0, 256, 32)
                k += 1
    return f


@pytest.mark.parametrize("noise", [False, True])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_corner_windows(ft, shift, noise):
    ctx = ft.Context(ft.default_limits(max_kp_per_image=512, max_map_points=64, max_batch_frames=1))
    f = corner_frame(40 + shift, shift, noise)
    want = oracle.run_frame(f)
    for batch in (False, True):
        df = ft.DeviceFrame(f, "cuda")
        if batch:
            ctx.ft_batch_wait(ctx.ft_batch_submit([df.job()]))
        else:
            df.run(ctx)
        torch.cuda.synchronize()
        compare_frame(df.results(), want)
