"""Batches of more than 64 jobs (a batch tile finds its job by comparing 64
prefix ends per load, in two steps beyond 64 jobs), some of them without
keypoints or map points: equal to the same frames through the single-frame
calls."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 64, 65, 128, 129, 300])
def test_jobs_equal_single_frames(ft, n):
    ctx = ft.Context(ft.default_limits(max_kp_per_image=256, max_map_points=1024, max_rows=256, max_batch_frames=n,
                                       max_inflight=1))
    base = [synth.tiny_clustered(100 + s, n_map=50 + 90 * s, n_kp=20 + 13 * s) for s in range(7)]
    base.append(dict(base[0], map={k: v[:0] for k, v in base[0]["map"].items()}))     # no map points
    frames = [ft.DeviceFrame(base[(i * 5) % len(base)], "cuda") for i in range(n)]
    want = []
    for f in base:
        d = ft.DeviceFrame(f, "cuda")
        d.run(ctx)
        torch.cuda.synchronize()
        want.append(d.results()["search"][0])
    t = ctx.ft_batch_submit([f.job() for f in frames])
    ctx.ft_batch_wait(t)
    for i, f in enumerate(frames):
        got, w = f.results()["search"][0], want[(i * 5) % len(base)]
        for k in ("mp_match", "mp_dist", "kp_match"):
            assert np.array_equal(got[k], w[k]), (i, k)
        assert got["n_matches"] == w["n_matches"], i
