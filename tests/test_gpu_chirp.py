"""2-D analyses at sides that run by chirp convolution (a prime factor above 5, 80 to 2048), against the oracle:
the first and last length of each convolution size, the lengths just outside, odd and even column
counts (real columns go in pairs), and mixtures with the other routes.

Error of a pass of length N, convolution length M: an FFT of length M is within 7 log2 M eps of its result in
the 2-norm (Higham, Accuracy and Stability of Numerical Algorithms, Theorem 24.2, whose constant is below 7).
With x chirped to a, b the chirp (2N - 1 values of modulus 1), A and B their transforms:
  |da| through B:  (1/M) sum |B| |dA| <= (1/M) |B|_2 |dA|_2 <= 7 log2 M eps sqrt(2N) |x|_2,
  |db| through A:  the same,
  the inverse:     7 log2 M eps |c|_2, |c|_2 <= |x|_1 |b|_2 <= sqrt(2N) |x|_1,
and the three chirp and table products add less than log2 M eps sqrt(2N) |x|_1 each, so
|dX| <= 24 log2 M sqrt(2N) eps |x|_1.  The first pass transforms x - m, m the mean to the nearest whole
number, and its 1-norm enters; so does the mixed-radix pass, which takes real columns in pairs too."""
import numpy as np
import pytest

from gpu_util import host, need_gpu, say, to_dev
from oracle import diagnostics as dg

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


@pytest.fixture(scope="module")
def ctx(lz):
    return lz.Context(0)


def _pass(n):
    """The factor of eps |x|_1 of a pass of length n by any route (4 (n + 2) for the others)."""
    m = 512
    while m < 2 * n - 1:
        m *= 2
    return max(4 * (n + 2), 24 * np.log2(m) * np.sqrt(2 * n))


def _dz(x):
    h, w = x.shape
    m = np.rint(x.astype(np.int64).sum() / x.size)
    return (_pass(h) + _pass(w)) * EPS * np.abs(x - m).sum()


def _power_tol(x):
    s1 = float(x.astype(np.float64).sum())
    dz = _dz(x)
    return 2 * s1 * dz + dz * dz + 4 * EPS * s1 * s1


def _acf_tol(x):
    h, w = x.shape
    n, xs = h * w, x.astype(np.int64)
    s1, s2 = int(xs.sum()), int((xs * xs).sum())
    den = float(n * s2 - s1 * s1)
    dz = _dz(x)
    return (2 * dz * n * np.sqrt(s2) + n * dz * dz + 2 * EPS * n * s2) / den + (_pass(h) + _pass(w) + 2) * EPS


SIZES = [(79, 82), (82, 83), (127, 129), (129, 1), (129, 2), (131, 3), (251, 257), (254, 7), (258, 33), (509, 511), (513, 16), (514, 1021),
         (1022, 5), (1023, 1024), (1025, 6), (1366, 77), (2039, 3), (2047, 130), (2049, 131), (4, 1009), (1, 683),
         (1000, 1006), (256, 262), (24, 45), (45, 7), (1000, 1), (96, 81), (125, 250)]


@pytest.mark.parametrize("h,w", SIZES)
def test_power_spectrum(lz, ctx, h, w):
    rng = np.random.default_rng(h * 11 + w)
    one = np.zeros((h, w), np.uint8)
    one[h // 3, w // 2] = 200
    for x in (rng.integers(0, 256, (h, w), dtype=np.uint8), rng.integers(0, 2, (h, w), dtype=np.uint8),
              np.full((h, w), 200, np.uint8), one):
        got = host(lz.power_spectrum_2d(ctx, to_dev(x.ravel()).view(h, w)))
        say(h, w)
        err = np.max(np.abs(got - dg.power_spectrum_2d(x)))
        assert err <= _power_tol(x), (h, w, err, _power_tol(x))


@pytest.mark.parametrize("h,w", SIZES)
def test_autocorrelation(lz, ctx, h, w):
    rng = np.random.default_rng(h * 13 + w)
    x = rng.integers(0, 256, (h, w), dtype=np.uint8)
    x[::3, ::2] = 255
    got = host(lz.autocorrelation_2d(ctx, to_dev(x.ravel()).view(h, w)))
    tol = _acf_tol(x)
    lags = [(0, 0), (h - 1, w - 1), (h // 2, w // 2), (min(3, h - 1), min(2, w - 1))]
    lags += [tuple(v) for v in rng.integers(0, [h, w], (8, 2))]
    for dx, dy in lags:
        want = dg.autocorrelation_2d_at(x, int(dx), int(dy))
        assert abs(got[dx, dy] - want) <= tol, (h, w, dx, dy, got[dx, dy], want, tol)
    const = np.full((h, w), 42, np.uint8)
    assert np.isnan(host(lz.autocorrelation_2d(ctx, to_dev(const.ravel()).view(h, w)))).all()
