"""Lag sums and autocorrelation past lag 256 of sequences of a few bytes, at every place within 16 bytes of memory (those that
do not reach the next multiple of 16 among them), against the oracle."""
import numpy as np
import pytest

from gpu_util import host, need_gpu, say, to_dev
from oracle import diagnostics as dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 7, 9, 14, 15, 16, 17, 33])
@pytest.mark.parametrize("L", [257, 4399, 16384])
def test_tiny(n, L):
    need_gpu()
    import paper_1201_3114_amd as lz

    ctx = lz.Context(0)
    rng = np.random.default_rng(n)
    for off in range(17):
        data = rng.integers(0, 256, off + n + 40, dtype=np.uint8)
        x = data[off:off + n].astype(np.int64)
        dev = to_dev(data)[off:off + n]
        say(n, L, off)
        got = host(lz.lag_sums(ctx, dev, L))
        want = np.zeros(L + 1, np.int64)
        for k in range(min(n, L + 1)):
            want[k] = (x[:n - k] * x[k:]).sum()
        assert np.array_equal(got, want), off
        r = host(lz.autocorrelation(ctx, dev, L))
        if (x == x[0]).all():
            assert np.isnan(r).all()
        else:
            # each coefficient is a quotient of a difference of terms up to S_0 + n m^2 <= 2 n 255^2 in a few roundings
            den = (x * x).sum() - x.sum() ** 2 / n
            tol = 16 * np.finfo(float).eps * 2 * n * 255 ** 2 / den
            exact = dg.autocorrelation(data[off:off + n], min(L, n))
            assert np.max(np.abs(r[:len(exact)] - exact)) <= tol and not r[n:].any(), off
