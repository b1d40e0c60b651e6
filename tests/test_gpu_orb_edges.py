"""ORB extraction at the edges of its kernels' tiles, against the oracle bit for
bit (angles within 1e-4 degrees): widths that are no multiple of four, the
widest image, levels with a handful of window pixels, the extreme thresholds;
keypoints at every allowed distance from the border, more of them than the
waves of one full launch hold."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu
SC = synth.scale_tables()


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_batch_frames=1, max_inflight=1))


@pytest.mark.parametrize("w,h,t", [(39, 39, 1), (41, 47, 20), (42, 200, 254), (1536, 43, 10), (1533, 50, 20), (763, 64, 1)])
def test_detection_at_odd_widths_and_thresholds(ft, ctx, w, h, t):
    rng = np.random.default_rng(w + h)
    img = rng.integers(0, 256, (h, w), dtype=np.uint8)
    img[h // 2, w // 2] = 255                  # a lone bright pixel on black: the largest score
    img[h // 2 - 4:h // 2 + 5, w // 2 - 4:w // 2 + 5] *= np.uint8(0)
    img[h // 2, w // 2] = 255
    pyr = oracle.pyramid(img, SC["inv_sf"])
    want = oracle.orb_detect(pyr, SC["sf"], t=t, edge=19)
    d = ft.DeviceOrb(pyr, capacity=max(want["count"], 1))
    for _ in range(2):
        d.detect(ctx, ft._scales(SC), threshold=t, edge=19)
    torch.cuda.synchronize()
    got = d.results()
    assert got["count"] == want["count"]
    for key in ("lx", "ly", "octave", "score", "x", "y"):
        assert np.array_equal(got[key], want[key][:got["count"]]), key
    assert np.array_equal(d.blurred.cpu().numpy(), oracle.orb_blur_pyramid(pyr))


@pytest.mark.parametrize("w,h,n", [(131, 93, 1), (131, 93, 700), (170, 151, 70001)])
def test_description_up_to_the_border(ft, ctx, w, h, n):
    img = np.random.default_rng(n).integers(0, 256, (h, w), dtype=np.uint8)
    pyr = oracle.pyramid(img, SC["inv_sf"])
    at = [(x, y, l) for l in range(8) for y in range(15, int(pyr["height"][l]) - 15)
          for x in range(15, int(pyr["width"][l]) - 15)]
    at = np.array(at, np.int64)
    pick = np.concatenate([np.arange(len(at) - 1, -1, -1)] * (n // len(at) + 1))[:n]   # the last level's corner first
    kp = {"lx": at[pick, 0].astype(np.int16), "ly": at[pick, 1].astype(np.int16), "octave": at[pick, 2].astype(np.uint8)}
    blurred = oracle.orb_blur_pyramid(pyr)
    pat = synth.orb_pattern()
    want = oracle.orb_describe(pyr, blurred, kp, pat)
    d = ft.DeviceOrb(pyr, capacity=n)
    d.blurred.copy_(torch.from_numpy(blurred))
    for k in kp:
        d.t[k].copy_(torch.from_numpy(kp[k]))
    d.t["count"].fill_(n)
    d.describe(ctx, pat)
    torch.cuda.synchronize()
    assert np.array_equal(d.t["desc"].cpu().numpy(), want["desc"])
    a = np.abs(d.t["angle"].cpu().numpy().astype(np.float64) - want["angle"].astype(np.float64))
    assert np.minimum(a, 360.0 - a).max() < 1e-4
