"""Search resolve at the edges of its workgroups (256 threads of one map point and
one keypoint in a call of up to 8192 keypoints, of four in a larger one and in a
batch) and of its groups of four, with more points than keypoints and fewer: equal
to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import compare_frame

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_kp_per_image=8200, max_map_points=4096, max_batch_frames=1, max_inflight=1))


@pytest.mark.parametrize("n_map", [1, 2, 3, 4, 5, 255, 256, 257, 1023, 1024, 1025, 1026, 1027, 2049])
@pytest.mark.parametrize("n_kp", [3, 256, 601])
def test_sizes_equal_oracle(ft, ctx, n_map, n_kp):
    f = synth.tiny_clustered(9, n_map=2100, n_kp=601)
    f["map"] = {k: v[:n_map] for k, v in f["map"].items()}
    f["left"] = {k: v[:n_kp] for k, v in f["left"].items()}
    for s in f["search"]:
        if s.get("preassigned") is not None:
            s["preassigned"] = s["preassigned"][:n_kp]
    want = oracle.run_frame(f)
    for batch in (False, True):
        df = ft.DeviceFrame(f, "cuda")
        if batch:
            ctx.ft_batch_wait(ctx.ft_batch_submit([df.job()]))
        else:
            df.run(ctx)
        torch.cuda.synchronize()
        compare_frame(df.results(), want)


@pytest.mark.parametrize("n_kp", [8191, 8192, 8193, 8195])
def test_many_keypoints_equal_oracle(ft, ctx, n_kp):
    f = synth.tiny_clustered(9, n_map=2100, n_kp=601)
    reps = -(-n_kp // 601)
    f["left"] = {k: np.ascontiguousarray(np.concatenate([v] * reps)[:n_kp]) for k, v in f["left"].items()}
    f["left"]["desc"][::3, 5] ^= 1
    for s in f["search"]:
        if s.get("preassigned") is not None:
            s["preassigned"] = np.concatenate([s["preassigned"]] * reps)[:n_kp]
    want = oracle.run_frame(f)
    df = ft.DeviceFrame(f, "cuda")
    df.run(ctx)
    torch.cuda.synchronize()
    compare_frame(df.results(), want)
