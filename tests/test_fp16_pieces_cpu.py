"""The error GEMM's fp16 operand split, modelled on the host: a value scaled
by a power of two, its row's (or layer's) maximum in [2^14, 2^15), is the sum of
fp16 values each rounded to nearest from the remainder so far, two for X and
three for D, and a product is summed from four of the six piece products.  These
checks pin the bounds the kernel's accuracy rests on: two pieces stay within
2^-23 |x| + 2^-25 of x (and are exact for most values), three within 2^-25, and
the product within what these and the one left out allow."""
import numpy as np


def pieces(x, n):
    r, out = np.asarray(x, dtype=np.float32), []
    for _ in range(n):
        h = r.astype(np.float16)
        out.append(h.astype(np.float64))
        exact = r.astype(np.float64) - out[-1]
        r = (r - h.astype(np.float32)).astype(np.float32)
        assert np.array_equal(r.astype(np.float64), exact)      # the remainder is exact in fp32
    return out


def _scaled(n, seed):
    """Values of one row, its maximum in [2^14, 2^15): from that down to fp16's subnormals and below."""
    rng = np.random.default_rng(seed)
    x = np.ldexp(rng.uniform(1.0, 2.0, n), rng.integers(-40, 15, n)) * rng.choice([-1.0, 1.0], n)
    x[0] = np.nextafter(np.float32(2.0 ** 15), np.float32(0))
    return x.astype(np.float32)


def test_split_error():
    x = _scaled(1 << 18, 1)
    f = x.astype(np.float64)
    h, lo = pieces(x, 2)
    assert np.all(np.isfinite(h)) and np.all(np.isfinite(lo))
    assert np.all(np.abs(h + lo - f) <= 2.0 ** -23 * np.abs(f) + 2.0 ** -25)
    assert np.all(np.abs(lo) <= 2.0 ** -11 * np.abs(f) + 2.0 ** -25)
    normal = np.abs(f) >= 2.0 ** -1                              # no piece of these is below fp16's spacing
    assert 0.7 < np.mean((h + lo == f)[normal]) < 0.8
    assert np.all(np.abs(sum(pieces(x, 3)) - f) <= 2.0 ** -25)


def test_four_products():
    d, x = _scaled(1 << 18, 2), _scaled(1 << 18, 3)
    dh, dm, dl = pieces(d, 3)
    xh, xl = pieces(x, 2)
    fd, fx = np.abs(d.astype(np.float64)), np.abs(x.astype(np.float64))
    four = dh * xh + dh * xl + dm * xh + dl * xh
    # left out: dm xl and dl xl, dm and xl at most 2^-11 of their values (a
    # remainder below half an ulp of 11 bits), dl 2^-22; and the splits' errors
    ed, ex = 2.0 ** -25, 2.0 ** -23 * fx + 2.0 ** -25
    bound = (2.0 ** -11 + 2.0 ** -22) * (fd + 2.0 ** -13) * (2.0 ** -11 * fx + 2.0 ** -25) * 1.001 \
        + ed * fx + ex * fd + ed * ex
    err = np.abs(four - d.astype(np.float64) * x)
    assert np.all(err <= bound)
    near = (fd > 2.0 ** 8) & (fx > 2.0 ** 8)                     # far above the spacing: 2^-22 + 2^-23 and a little
    assert np.all(err[near] <= 2.0 ** -21 * (fd * fx)[near])
