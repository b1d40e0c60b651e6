"""Search by projection with level windows far wider than the octaves: every
keypoint octave passes, so every window at least that wide gives the oracle's
matches, for the record-dealt search and for lane groups, single-frame and
batched."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import compare_frame

pytestmark = pytest.mark.gpu

INT_MAX = 2**31 - 1


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_kp_per_image=2048, max_map_points=4096, max_batch_frames=1))


def frame(lo, hi):
    f = synth.tiny_clustered(77, n_map=1500, n_kp=700)
    f["search_params"] = dict(f["search_params"], level_lo=lo, level_hi=hi, th=6.0)
    return f


@pytest.mark.parametrize("lanes", [1, 4])
@pytest.mark.parametrize("lo,hi", [(7, 7), (16, 232), (17, 0), (17, 240), (1, 233), (240, 1), (255, 256), (300, 65536),
                                   (0, INT_MAX - 7), (INT_MAX, INT_MAX)])
def test_wide_windows_equal_oracle(ft, ctx, lo, hi, lanes):
    f = frame(lo, hi)
    # (predicted levels and octaves are 0 .. 7; the oracle adds without a check for overflow)
    want = oracle.run_frame(frame(min(lo, 100), min(hi, 100)))
    assert want["search"][0]["n_matches"] > 50
    ctx.ft_set_shapes(8, lanes)
    for batch in (False, True):
        df = ft.DeviceFrame(f, "cuda")
        if batch:
            ctx.ft_batch_wait(ctx.ft_batch_submit([df.job()]))
        else:
            df.run(ctx)
        torch.cuda.synchronize()
        compare_frame(df.results(), want)
    levels = np.unique(f["left"]["octave"][want["search"][0]["mp_match"][want["search"][0]["mp_match"] >= 0]])
    assert len(levels) > 3


@pytest.mark.parametrize("rows", [160, 1100])
@pytest.mark.parametrize("window", [7, 255, 256, 65536, INT_MAX - 3, INT_MAX])
def test_wide_stereo_windows_equal_oracle(ft, window, rows):
    """The stereo level window: row bins per level (8 x 160) and one for every level."""
    ctx = ft.Context(ft.default_limits(max_kp_per_image=512, max_map_points=512, max_rows=2048, max_batch_frames=1,
                                       max_inflight=1))
    f = synth.tiny_pinhole(55, n_kp=400)
    f["stereo_cam"] = dict(f["stereo_cam"], rows=rows)
    want = oracle.run_frame(dict(f, stereo_params=dict(f["stereo_params"], level_window=7)))
    assert want["stereo"]["n_matches"] > 50
    for batch in (False, True):
        df = ft.DeviceFrame(dict(f, stereo_params=dict(f["stereo_params"], level_window=window)), "cuda")
        if batch:
            ctx.ft_batch_wait(ctx.ft_batch_submit([df.job()]))
        else:
            df.run(ctx)
        torch.cuda.synchronize()
        compare_frame(df.results(), want)
