"""Fisheye all-pairs search at the edges of its tiles (16 targets a column block,
four waves, four tiles in flight per wave; 32 queries per workgroup), with
descriptors of no and of all bits and with ties: equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import compare_frame

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_kp_per_image=1024, max_map_points=512, max_batch_frames=1))


def overlap(x, count):
    """A closed interval of x that holds the `count` smallest values."""
    return np.array([np.min(x) - 1, np.sort(x)[count - 1]], np.float32)


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("targets,queries", [(2, 1), (3, 31), (15, 32), (16, 33), (17, 64), (63, 65), (64, 97),
                                             (65, 129), (193, 30), (240, 100), (255, 200), (256, 256), (257, 1),
                                             (271, 300), (449, 128), (512, 90), (513, 511), (767, 513)])
def test_sizes(ft, ctx, targets, queries, batch):
    f = synth.tiny_fisheye(900 + targets, n_kp=820, n_map=100)
    f["search"] = f["search"][:1]
    r = np.random.default_rng(targets)
    for side, step in (("left", 9), ("right", 7)):
        d = f[side]["desc"]
        d[0::step] = 0
        d[1::step] = 255
        d[2::step] = d[2]
        d[3::step] ^= (r.random(d[3::step].shape) < 0.02).astype(d.dtype)
        x = f[side]["x"]
        x += np.arange(len(x), dtype=np.float32) * np.float32(1e-3)    # distinct, so that counts are exact
    nl, nr = min(queries, f["left"]["x"].size), min(targets, f["right"]["x"].size)
    f["stereo_cam"]["overlap_left"] = overlap(f["left"]["x"], nl)
    f["stereo_cam"]["overlap_right"] = overlap(f["right"]["x"], nr)
    want = oracle.run_frame(f)
    assert (want["stereo"]["stats"]["Q"], want["stereo"]["stats"]["T"]) == (nl, nr)
    df = ft.DeviceFrame(f, "cuda")
    if batch:
        ctx.ft_batch_wait(ctx.ft_batch_submit([df.job()]))
    else:
        df.run(ctx)
    torch.cuda.synchronize()
    compare_frame(df.results(), want)
