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


def test_ticks_do_not_mix_layouts_beside_other_work(lz):
    """40,000 chains of 256 bytes are 16 ticks of a lane per chain.  Mixed ticks take 18 or more: most chains get 13 bytes in
    each.  Beside short messages on another stream at most the first two are mixed."""
    import time

    import torch

    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    ctx, other = lz.Context(0), lz.Context(0, lz.params(n_it=160))
    per = simds * 2000 // 1024
    P = [torch.randint(0, 256, (256 * per,), dtype=torch.uint8, device="cuda") for _ in range(20)]
    want = [ctx.encrypt(p, b"tick") for p in P]
    out = [torch.empty(256 * per + 24, dtype=torch.uint8, device="cuda") for _ in P]
    msg = torch.zeros(simds * 64 * 256, dtype=torch.uint8, device="cuda")
    msg_out = torch.empty(len(msg) + 24, dtype=torch.uint8, device="cuda")
    msg_want = other.encrypt(msg, b"message")

    def burst(beside):
        srv, s1 = lz.Server(ctx, hbm_budget=1 << 30), torch.cuda.Stream()
        for o in out:
            o.zero_()
        torch.cuda.synchronize()
        for _ in range(beside):
            other.encrypt(msg, b"message", out=msg_out, stream=s1)
        srv.submit_many(list(range(20)), [0] * 20, [b"tick"] * 20, [p.data_ptr() for p in P], [len(p) for p in P],
                        [o.data_ptr() for o in out], [lz.now_ns()] * 20)
        n, end = 0, time.monotonic() + 30
        while n < 20 and time.monotonic() < end:
            n += len(srv.poll(20, 10))
        assert n == 20
        ticks = srv.stats()["ticks"]
        srv.close()
        for o, x in zip(out, want):
            assert torch.equal(o, x)
        return ticks

    alone = burst(0)
    say("alone", alone)
    assert alone >= 18
    beside = []
    for _ in range(12):  # until a stream whose hardware queue is not the server's
        beside.append(burst(60))
        assert torch.equal(msg_out, msg_want)
        if beside[-1] <= 17:
            break
    say("beside", beside)
    assert beside[-1] <= 17
    torch.cuda.synchronize()
    assert lz.unit_waves(ctx) == 0


@pytest.mark.parametrize("over,rounds", [(1, False), (256, True), (64 * 256 + 1, True)])
def test_a_short_last_block_needs_no_rounds(lz, streams, over, rounds):
    """A message of one block over a wave per SIMD: where that block is short, it runs beside the others in one launch, whose
    waves are one more workgroup than a round's."""
    import torch

    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    n = simds * 64 * 256 + over
    ctx = lz.Context(0)
    P = to_dev(np.random.default_rng(over).integers(0, 256, n, dtype=np.uint8))
    out = torch.empty(n + 24, dtype=torch.uint8, device="cuda")
    seen = samples(lz, ctx, lambda s: ctx.encrypt(P, b"last", out=out, stream=s), *streams)
    say(over, max(seen))
    assert max(seen) == (simds if rounds else simds + 4)
    assert torch.equal(ctx.decrypt(out, b"last"), P)
    # the same blocks as in a message without the last ones
    assert torch.equal(ctx.encrypt(P[:-over], b"last")[:-24], out[:n - over])
