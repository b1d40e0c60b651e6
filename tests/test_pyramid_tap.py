"""The pyramid build's tap arithmetic, over sizes up to the largest it accepts:
the quotient from a binary32 reciprocal that is one unit in the last place off
either way, corrected by at most one with a remainder kept modulo 2^32, equals the
exact floor(256 num / den), and so do the pixel and weight it gives."""
import numpy as np
import pytest

MAX_W, MAX_H = 1536, 4096


def taps(n_in, n_out, ulps):
    """Pixel and weight of every output index, as the kernel computes them with a
    reciprocal `ulps` units in the last place from the rounded one."""
    x = np.arange(n_out, dtype=np.int64)
    num = (2 * x + 1) * n_in - n_out
    den = 2 * n_out
    assert num.max() < 2**26 and den <= 2**13
    rcp = np.float32(1) / np.float32(den)
    for _ in range(abs(ulps)):
        rcp = np.nextafter(rcp, np.float32(np.inf if ulps > 0 else 0))
    f = np.floor((num.astype(np.float32) * np.float32(256)) * rcp)
    t = np.maximum(f, 0).astype(np.int64)
    r = ((num << 8) - t * den) & 0xFFFFFFFF
    r = np.where(r >= 2**31, r - 2**32, r)                   # the difference as a signed 32-bit value
    t = np.where(r < 0, t - 1, np.where(r >= den, t + 1, t))
    q = t >> 8
    end = q >= n_in - 1
    return np.where(num <= 0, 0, np.where(end, n_in - 1, q)), np.where((num <= 0) | end, 0, t & 255)


@pytest.mark.parametrize("limit", [MAX_W, MAX_H])
def test_taps_are_exact(limit):
    rng = np.random.default_rng(limit)
    sizes = [(n, m) for n in (2, 3, 15, 16, 17, 752, limit - 1, limit) for m in {1, 2, n // 3 + 1, n // 2 + 1, n - 1, n} if m <= n]
    sizes += [(limit, int(round(limit / f ** l))) for f in (1.05, 1.2, 1.5, 2.0) for l in range(1, 8)]
    for n in rng.integers(2, limit + 1, 400):
        sizes.append((int(n), int(rng.integers(1, n + 1))))
    for n_in, n_out in sizes:
        x = np.arange(n_out, dtype=np.int64)
        num = np.maximum((2 * x + 1) * n_in - n_out, 0)
        t = 256 * num // (2 * n_out)
        end = (t >> 8) >= n_in - 1
        want = np.where(end, n_in - 1, t >> 8), np.where(end, 0, t & 255)
        for ulps in (-1, 0, 1):
            got = taps(n_in, n_out, ulps)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (n_in, n_out, ulps)
