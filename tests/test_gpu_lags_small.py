"""The histogram, lag sums and coefficients where a launch has one workgroup (to 16 KiB) and two, and the coefficients
past lag 256, where each workgroup of the correction kernel needs lag 0 and the byte total: exact counts and sums,
coefficients against extended precision, calls repeated (the merge buffer is left clear)."""
import numpy as np
import pytest

from gpu_util import host, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def sums(x, L):
    v = x.astype(np.int64)
    return np.array([int((v[: len(v) - k] * v[k:]).sum()) if k < len(v) else 0 for k in range(L + 1)])


def coefficients(x, L):
    n, ld = len(x), np.longdouble
    d = x.astype(ld) - x.astype(ld).mean()
    return np.array([(d[: n - k] * d[k:]).sum() if k < n else ld(0) for k in range(L + 1)]) / (d * d).sum()


@pytest.mark.parametrize("n,L", [(1, 0), (2, 3), (100, 256), (16383, 31), (16384, 256), (16385, 256), (32769, 32),
                                 (300, 300), (5000, 257), (32769, 1000), (20001, 4500), (9000, 16384), (70001, 5000),
                                 (600000, 520)])
@pytest.mark.parametrize("skip", [0, 3], ids=["aligned", "odd"])
def test_against_exact(lz, n, L, skip):
    x = np.random.default_rng(n + L).integers(0, 256, n + skip, dtype=np.uint8)
    dev, x = to_dev(x)[skip:], x[skip:]
    ctx = lz.Context(0)
    want = sums(x, L)
    for _ in range(2):
        assert np.array_equal(host(lz.histogram(ctx, dev)), np.bincount(x, minlength=256))
        assert np.array_equal(host(lz.lag_sums(ctx, dev, L)), want)
        r = host(lz.autocorrelation(ctx, dev, L))
        if n == 1:
            assert np.isnan(r).all()
            continue
        # the numerator's terms are at most S_0, 2 S_0 and S_0, the denominator's S_0 each, with up to six roundings
        # in each: relative to the denominator
        den = want[0] - int(x.sum(dtype=np.int64)) ** 2 / n
        assert np.abs(r - coefficients(x, L)).max() <= 2.0 ** -53 * 40 * want[0] / den
    ctx.close()


@pytest.mark.parametrize("n,L", [(64, 10), (16384, 256), (900, 300), (0, 5), (0, 700)])
def test_no_coefficient(lz, n, L):
    ctx = lz.Context(0)
    assert np.isnan(host(lz.autocorrelation(ctx, to_dev(np.full(n, 77, np.uint8)), L))).all()
    ctx.close()
