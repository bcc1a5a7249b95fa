"""entropy(): its one number reaches the host in a pinned word of the context.  The value is seen while the call polls,
or, where work ahead of it on the stream takes longer than that, after the runtime's own wait; threads take turns."""
import threading
from contextlib import closing

import numpy as np
import pytest

from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu

# 256 terms -p log2 p <= 0.54 of two roundings and a logarithm of 2 ulp each, and 256 additions to at most 8
TOL = 256 * (4 * 0.54 + 8) * 2.0 ** -53


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def entropy64(data):
    p = np.bincount(data, minlength=256) / data.size
    p = p[p > 0]
    return float(-(p * np.log2(p)).sum())


@pytest.mark.parametrize("ahead", [0, 64 * 1024], ids=["idle", "13ms_ahead"])
def test_value_after_the_work_ahead(lz, ahead):
    import torch

    data = np.random.default_rng(3).integers(0, 200, 70001, dtype=np.uint8)
    dev, msg = to_dev(data), to_dev(np.zeros(ahead, np.uint8))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with closing(lz.Context(0)) as ctx, torch.cuda.stream(s):
        for _ in range(3):
            if ahead:
                ctx.encrypt(msg, b"entropy", stream=s)
            assert abs(lz.entropy(ctx, lz.histogram(ctx, dev, stream=s), stream=s) - entropy64(data)) <= TOL


def test_threads_on_one_context(lz):
    import torch

    done = []

    def work(ctx, hist, want):
        s = torch.cuda.Stream()
        done.append(all(abs(lz.entropy(ctx, hist, stream=s) - want) <= TOL for _ in range(50)))

    with closing(lz.Context(0)) as ctx:
        data = [np.random.default_rng(i).integers(0, 2 + 50 * i, 5000, dtype=np.uint8) for i in range(4)]
        hists = [lz.histogram(ctx, to_dev(d)) for d in data]
        torch.cuda.synchronize()
        threads = [threading.Thread(target=work, args=(ctx, h, entropy64(d))) for h, d in zip(hists, data)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert done == [True] * 4
