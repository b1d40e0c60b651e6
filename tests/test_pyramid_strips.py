"""The pyramid build's strips, restated on the host: every output byte of
every level is written once and equals the oracle's, each dword a lane reads
holds at least one byte of the image, and the byte windows of the four columns
fit the dword pair the kernel picks for the level's scale.

The restatement follows the kernel's rules: strips of 256 columns by 2^r rows;
kNear / kMid / kFar by the level's scale (up to 2, 10/3, 11/3), kAny beyond, for
images under 16 columns and for strips that reach the image's last bytes."""
import numpy as np
import pytest

import oracle
import synth

SC = synth.scale_tables()


def _taps(x, n_in, n_out):
    num = (2 * x + 1) * n_in - n_out
    t = np.where(num <= 0, 0, 256 * num // (2 * n_out))
    q, w = t >> 8, t & 255
    end = q >= n_in - 1
    return np.where(end, n_in - 1, q), np.where(end, 0, w)


def _strip(buf, src, W, H, pitch, wl, hl, bx, ylo, yhi, reach, n_bytes):
    """Output rows of one strip [yhi - ylo, 256], computed from the bytes the
    lanes read; checks the reads."""
    lane = np.arange(64)
    x = 256 * bx + 4 * lane
    x0, a = zip(*[_taps(np.minimum(x + k, wl - 1), W, wl) for k in range(4)])
    yt, b = _taps(np.arange(ylo, yhi), H, hl)

    def pairs(y):
        row = src + y * pitch
        if reach == "any":
            return [(buf[row + x0[k]], buf[row + np.minimum(x0[k] + 1, W - 1)]) for k in range(4)]
        sh = row & 3
        off = row - sh + ((x0[0] + sh) & ~3)
        for i in range(4):   # bytes [off + 4 i, off + 4 i + 4) meet [src, src + n_bytes)
            assert ((off + 4 * i + 3 >= src) & (off + 4 * i < src + n_bytes)).all(), (W, H, wl, hl, bx, y)
        al = (x0[0] + sh) & 3
        out = []
        for k in range(4):
            first = 8 if reach == "far" and k == 3 else 4 if reach != "near" and k >= 2 else 0
            o = x0[k] - x0[0]
            live = x + k < wl
            assert ((o[live] >= first) & (o[live] + 1 <= first + 7)).all(), (reach, W, wl, k)
            assert (al[live] + o[live] + 1 <= 15).all() or (a[k][live][al[live] + o[live] + 1 > 15] == 0).all()
            out.append((buf[off + al + o], buf[np.minimum(off + al + o + 1, off + 15)]))
        return out

    res = np.zeros((yhi - ylo, 256), np.int64)
    for r in range(yhi - ylo):
        top, bot = pairs(yt[r]), pairs(min(yt[r] + 1, H - 1))
        for k in range(4):
            h = [(256 - a[k]) * p.astype(np.int64) + a[k] * q.astype(np.int64) for p, q in (top[k], bot[k])]
            res[r, k::4] = ((256 - b[r]) * h[0] + b[r] * h[1] + 32768) >> 16
    return res


@pytest.mark.parametrize("W,H,pitch,shift,r", [(752, 37, 752, 0, 2), (515, 61, 517, 1, 3), (16, 16, 16, 3, 2), (17, 300, 17, 2, 4),
                                              (257, 40, 260, 0, 2), (1281, 30, 1283, 3, 4), (15, 64, 64, 0, 3),
                                              (309, 64, 309, 1, 2), (1536, 9, 1536, 2, 2)])
def test_strips_write_the_oracle_pyramid(W, H, pitch, shift, r):
    img = np.random.default_rng(W + H).integers(0, 256, (H, W), dtype=np.uint8)
    src, n_bytes = 64 + shift, (H - 1) * pitch + W
    buf = np.full(src + n_bytes + 64, 0x5A, np.uint8)
    for y in range(H):
        buf[src + y * pitch: src + y * pitch + W] = img[y]
    want = oracle.pyramid(img, SC["inv_sf"])
    for l in range(1, 8):
        wl, hl = int(want["width"][l]), int(want["height"][l])
        ref = want["data"][int(want["offset"][l]):][:wl * hl].reshape(hl, wl)
        got = np.full((hl, wl), -1, np.int64)
        for bx in range(-(-wl // 256)):
            for ylo in range(0, hl, 1 << r):
                yhi = min(ylo + (1 << r), hl)
                corner = yhi >= hl - 1 and 256 * (bx + 1) + 20 >= wl
                reach = ("any" if corner or W < 16 or 3 * W > 11 * wl else "near" if W <= 2 * wl else
                         "mid" if 3 * W <= 10 * wl else "far")
                s = _strip(buf, src, W, H, pitch, wl, hl, bx, ylo, yhi, reach, n_bytes)
                n = min(256, wl - 256 * bx)
                assert (got[ylo:yhi, 256 * bx:256 * bx + n] == -1).all()
                got[ylo:yhi, 256 * bx:256 * bx + n] = s[:, :n]
        assert np.array_equal(got, ref), (W, H, l)
