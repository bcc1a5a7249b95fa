"""2-D analyses whose four passes are all direct DFTs on the matrix cores, in tiles of 64 x 64 outputs: both sides past the chirp
convolution's 2048, with a prime factor above 5, and tiles enough for every compute unit in each pass (the passes over
bytes, over doubles, and those that write power and correlation).

Error of a pass of length N: a sum of N complex products with a factor of modulus 1 in fused multiply-adds is off by at
most 2 N eps sum|x| in each component (the factors' own errors add a few eps), so |dZ| <= 4 (h + w + 4) eps S after
two passes, S the 1-norm of what goes in: x - m, m the mean to the nearest whole number."""
import numpy as np
import pytest

from gpu_util import host, need_gpu, say, to_dev
from oracle import diagnostics as dg

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _dz(x):
    m = np.rint(x.astype(np.int64).sum() / x.size)
    return 4 * (sum(x.shape) + 4) * EPS * np.abs(x - m).sum()


@pytest.mark.parametrize("h,w", [(2053, 2063), (2059, 4099)])
def test_direct(h, w):
    need_gpu()
    import torch

    import paper_1201_3114_amd as lz

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert (h // 2 // 64 + 1) * (w // 64 + 1) >= cus and h * w <= 1 << 24
    rng = np.random.default_rng(h)
    x = rng.integers(0, 256, (h, w), dtype=np.uint8)
    x[::4, ::7] = 255
    ctx = lz.Context(0)
    s1, s2, n = int(x.astype(np.int64).sum()), int((x.astype(np.int64) ** 2).sum()), h * w
    dz = _dz(x)
    say(h, w)
    got = host(lz.power_spectrum_2d(ctx, to_dev(x.ravel()).view(h, w)))
    tol = 2 * s1 * dz + dz * dz + 4 * EPS * s1 * s1
    assert np.max(np.abs(got - dg.power_spectrum_2d(x))) <= tol
    got = host(lz.autocorrelation_2d(ctx, to_dev(x.ravel()).view(h, w)))
    den = float(n * s2 - s1 * s1)
    tol = (2 * dz * n * np.sqrt(s2) + n * dz * dz + 2 * EPS * n * s2) / den + 4 * (h + w + 6) * EPS
    lags = [(0, 0), (1, 0), (0, 1), (4, 7), (h // 2, w // 2), (h // 2 + 1, 3), (h - 1, w - 1), (h - 4, 7)]
    lags += [tuple(v) for v in rng.integers(0, [h, w], (4, 2))]
    for dx, dy in lags:
        want = dg.autocorrelation_2d_at(x, int(dx), int(dy))
        assert abs(got[dx, dy] - want) <= tol, (dx, dy, got[dx, dy], want, tol)
    # an even matrix: A[-dx][-dy] = A[dx][dy], bit for bit for the mirrored rows
    assert np.array_equal(got[1:], got[:0:-1, np.r_[0, w - 1:0:-1]])
