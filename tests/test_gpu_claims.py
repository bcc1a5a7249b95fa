"""The device's count of waves in flight, by which launches decide how many lanes a chain gets: calls that run in
rounds hold their claim between the rounds, and nothing is left counted at rest."""
import numpy as np
import pytest

from gpu_util import host, need_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def samples(lz, ctx, run, s1, s2):
    """The count, read on stream s2 again and again while run(s1)'s work runs."""
    import torch

    torch.cuda.synchronize()
    done = torch.cuda.Event()
    run(s1)
    done.record(s1)
    seen = []
    while not done.query():
        seen.append(lz.unit_waves(ctx, stream=s2))
    torch.cuda.synchronize()
    assert lz.unit_waves(ctx) == 0
    return seen


@pytest.fixture(scope="module")
def streams(lz):
    """Two streams whose work overlaps: streams may share one of the process's hardware queues."""
    import torch

    ctx = lz.Context(0)
    P = torch.zeros(3_000_000, dtype=torch.uint8, device="cuda")
    s1 = torch.cuda.Stream()
    for _ in range(16):
        s2 = torch.cuda.Stream()
        if sum(w > 0 for w in samples(lz, ctx, lambda s: ctx.encrypt(P, b"queue", stream=s), s1, s2)) >= 20:
            return s1, s2
    pytest.fail("no two streams overlap")


# a mix plan (two layouts), a segment plan (more than one wave per SIMD)
@pytest.mark.parametrize("n", [6 << 20, 20_000_000])
@pytest.mark.parametrize("kind", ["message", "batch"])
def test_rounds_hold_their_claim(lz, streams, n, kind):
    import torch

    ctx = lz.Context(0)
    P = to_dev(np.random.default_rng(n).integers(0, 256, n, dtype=np.uint8))
    out = torch.empty(n + 24, dtype=torch.uint8, device="cuda")
    want = host(ctx.encrypt(P, b"claims"))
    if kind == "batch":
        b = lz.Batch(ctx, False, [n], [b"claims"], P, [0], out, [0])
        run = lambda s: b.encrypt(stream=s)
    else:
        run = lambda s: ctx.encrypt(P, b"claims", out=out, stream=s)
    for _ in range(8):
        out.zero_()
        seen = samples(lz, ctx, run, *streams)
        busy = [i for i, w in enumerate(seen) if w]
        say(kind, n, len(seen), len(busy))
        assert len(busy) >= 20  # of some 20 ms
        assert busy == list(range(busy[0], busy[-1] + 1)), [seen[i] for i in range(busy[0], busy[-1] + 1)].index(0)
        assert np.array_equal(host(out), want)
