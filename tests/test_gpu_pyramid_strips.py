"""The pyramid build's strips on the device, byte for byte against the oracle:
the strip heights that a launch picks by its number of images (4 rows up to 2
images, 8 up to 16, 16 beyond), images of odd widths, padded rows and rows that
begin at any byte; and levels smaller by any scale, at full strip width, so that
every way of reading the four columns' taps runs: scales up to 2, up to 10/3, up
to 11/3, and beyond, where each column has a dword pair of its own."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

SC = synth.scale_tables()
SIZES = [(752, 480, 752), (515, 61, 517), (257, 40, 260), (1281, 30, 1283), (1536, 96, 1536), (309, 64, 309),
         (101, 67, 101), (17, 300, 17), (15, 64, 64), (255, 129, 260)]


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_kp_per_image=256, max_map_points=256, max_batch_frames=24, max_inflight=1))


def on_device(img, pitch, shift):
    """The image's rows `pitch` bytes apart from byte `shift` of an allocation
    that ends with the last row."""
    H, W = img.shape
    buf = np.full(shift + pitch * (H - 1) + W, 0x5A, np.uint8)
    for y in range(H):
        buf[shift + y * pitch: shift + y * pitch + W] = img[y]
    return torch.from_numpy(buf).cuda()


def check(got, img, inv_sf, tag):
    want = oracle.pyramid(img, inv_sf)["data"]
    bad = np.nonzero(got != want)[0]
    assert bad.size == 0, f"{tag}: {bad.size} bytes differ, first at {bad[:8].tolist()}"


@pytest.mark.parametrize("n_jobs", [1, 2, 8, 9, 20])
def test_batches_of_images(ft, ctx, n_jobs):
    base = synth.tiny_pinhole(5)
    for side in ("left", "right"):
        base[side] = {k: v[:0] for k, v in base[side].items()}
    base["map"] = {k: v[:0] for k, v in base["map"].items()}
    base["search"] = []
    rng = np.random.default_rng(n_jobs)
    frames, jobs, images = [], [], []
    for i in range(n_jobs):
        W, H, pitch = SIZES[(3 * i + n_jobs) % len(SIZES)]
        df = ft.DeviceFrame(base, "cuda", build_pyramids=True)
        job = df.job()
        for side in ("left", "right"):
            img = rng.integers(0, 256, (H, W), dtype=np.uint8)
            shift = int(rng.integers(0, 4))
            src = on_device(img, pitch, shift)
            lay, n = ft.pyramid_layout(W, H, df.scales)
            out = torch.full((n + 3,), 0xA5, dtype=torch.uint8, device="cuda")
            lay.data = out.data_ptr() + shift                   # (the pyramid begins at any byte too)
            setattr(job, "image_" + side, ft.ft_image(src.data_ptr() + shift, W, H, pitch))
            setattr(job, "pyr_" + side, lay)
            images.append((img, src, out, shift, n, (i, side, W, H, pitch, shift)))
        frames.append(df)
        jobs.append(job)
    for _ in range(2):
        ctx.ft_batch_wait(ctx.ft_batch_submit(jobs))
    torch.cuda.synchronize()
    for img, src, out, shift, n, tag in images:
        host = out.cpu().numpy()
        check(host[shift:shift + n], img, SC["inv_sf"], tag)
        assert (host[:shift] == 0xA5).all() and (host[shift + n:] == 0xA5).all(), tag


@pytest.mark.parametrize("factor", [1.0, 1.05, 1.2, 1.25, 1.45, 1.52, 1.9, 2.0])
@pytest.mark.parametrize("W,H,pitch,shift", [(1536, 300, 1536, 0), (1281, 719, 1283, 3), (509, 511, 512, 1),
                                             (131, 4096, 131, 2)])
def test_scale_factors(ft, ctx, factor, W, H, pitch, shift):
    sc = synth.scale_tables(factor=factor)
    scales = ft._scales(sc)
    lay, n = ft.pyramid_layout(W, H, scales)
    img = np.random.default_rng(W + H).integers(0, 256, (H, W), dtype=np.uint8)
    src = on_device(img, pitch, shift)
    out = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")
    lay.data = out.data_ptr()
    ctx.ft_build_pyramid(ft.ft_image(src.data_ptr() + shift, W, H, pitch), scales, lay)
    torch.cuda.synchronize()
    check(out.cpu().numpy(), img, sc["inv_sf"], (factor, W, H))


@pytest.mark.parametrize("W", [64, 65, 66, 76, 77, 78, 92, 93])
@pytest.mark.parametrize("H,pad,shift", [(9, 0, 0), (131, 3, 1), (1000, 0, 3)])
def test_narrow_levels(ft, ctx, W, H, pad, shift):
    """Images and levels of 64 columns (a column per lane) and of one more (four)."""
    scales = ft._scales(SC)
    lay, n = ft.pyramid_layout(W, H, scales)
    img = np.random.default_rng(W * H).integers(0, 256, (H, W), dtype=np.uint8)
    src = on_device(img, W + pad, shift)
    out = torch.full((n + 1,), 0xA5, dtype=torch.uint8, device="cuda")
    lay.data = out.data_ptr()
    ctx.ft_build_pyramid(ft.ft_image(src.data_ptr() + shift, W, H, W + pad), scales, lay)
    torch.cuda.synchronize()
    host = out.cpu().numpy()
    check(host[:n], img, SC["inv_sf"], (W, H))
    assert host[n] == 0xA5
