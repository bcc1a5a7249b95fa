"""Messages, stream updates and batches that run by a launch plan, against the oracle bit for bit.  Each case first asks the
library for its plan, so that none of them runs the ordinary launch unnoticed: mix plans of every pair of layouts
(1 and 4, 4 and 16, the fused map's 1 and 16 lanes per chain), of long blocks too; segment plans whose last segment is
shorter, with one to five full waves per SIMD before them, and with partial blocks among the planned waves."""
import numpy as np
import pytest

import oracle
from gpu_util import ORACLE_THREADS, host, need_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


@pytest.fixture(scope="module")
def simds(lz):
    import torch

    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


def mix_of(lz, simds, prm, chains):
    p = lz.unit_plan(lz.params(**prm), simds, chains)
    return tuple(p.mix_lanes) if p.mix_rounds else None


def both_ways(lz, prm, P):
    ctx = lz.Context(0, lz.params(**prm))
    C = ctx.encrypt(to_dev(P), b"plan")
    want = oracle.encrypt(b"plan", P, nthreads=ORACLE_THREADS, **prm)
    assert np.array_equal(host(C), want)
    assert np.array_equal(host(ctx.decrypt(C, b"plan")), P)
    bad = C.clone()
    bad[len(P) // 2] ^= 1
    with pytest.raises(lz.IntegrityError):
        ctx.decrypt(bad, b"plan")


# chains per SIMD, and a few more
MIX = [("euler", 4, 70, 256, 1000, (4, 16)), ("euler", 5, 3, 128, 1000, (4, 16)), ("euler", 6, -7, 250, 3000, (4, 16)),
       ("euler", 17, 1, 61, 640, (1, 4)), ("euler", 30, -1, 64, 1000, (1, 4)), ("euler", 36, 5, 128, 640, (1, 4)),
       ("euler_fma", 4, 1, 256, 640, (1, 16)), ("euler_fma", 5, -9, 128, 1000, (1, 16)), ("euler_fma", 7, 33, 100, 3000, (1, 16)),
       ("rk4", 4, 11, 250, 150, (4, 16)), ("rk4", 5, 0, 100, 640, (4, 16)), ("rk4", 6, -3, 100, 640, (4, 16)),
       ("rk4", 17, 2, 61, 150, (1, 4)), ("rk4", 30, 1, 61, 150, (1, 4)),
       ("euler", 4, 100, 1000, 300, (4, 16)), ("euler", 20, 3, 1000, 300, (1, 4)), ("euler", 5, 3, 4096, 100, (4, 16))]


@pytest.mark.parametrize("integ,per,more,block,n_it,lanes", MIX)
def test_mix_messages(lz, simds, integ, per, more, block, n_it, lanes):
    prm = dict(n_it=n_it, block_len=block, integrator=integ)
    chains = per * simds + more
    assert mix_of(lz, simds, prm, chains) == lanes
    rng = np.random.default_rng(chains)
    say(integ, chains, block, n_it)
    both_ways(lz, prm, rng.integers(0, 256, chains * block - min(block - 1, 11), dtype=np.uint8))


@pytest.mark.parametrize("integ,per,block,n_it,lanes", [
    ("euler", 4.5, 128, 1000, (4, 16)), ("euler_fma", 4.5, 128, 1000, (1, 16)), ("rk4", 4.5, 100, 640, (4, 16)),
    ("rk4", 18, 61, 150, (1, 4)), ("euler", 20, 61, 640, (1, 4))])
def test_mix_stream_updates(lz, simds, integ, per, block, n_it, lanes):
    """A first update that leaves its last block half done, a short one inside that block, and one that completes it."""
    prm = dict(n_it=n_it, block_len=block, integrator=integ)
    full = int(per * simds)
    for chains in (full + 1, full + 2):  # whole blocks and a tail; head, whole blocks and tail
        assert mix_of(lz, simds, prm, chains) == lanes
    cuts = [0, full * block + 13, full * block + 20, (2 * full + 1) * block + 9]
    rng = np.random.default_rng(full)
    P = rng.integers(0, 256, cuts[-1], dtype=np.uint8)
    want = oracle.encrypt(b"plan", P, nthreads=ORACLE_THREADS, **prm)
    ctx = lz.Context(0, lz.params(**prm))
    for decrypt in (False, True):
        src = to_dev(want[:len(P)] if decrypt else P)
        st = lz.Stream(ctx, decrypt, b"plan")
        say(integ, full, decrypt)
        body = np.concatenate([host(st.update(src[a:e].clone())) for a, e in zip(cuts, cuts[1:])])
        if decrypt:
            assert np.array_equal(body, P)
            st.finish(to_dev(want[len(P):]))  # raises if the tag differs
        else:
            assert np.array_equal(np.concatenate([body, host(st.finish())]), want)
        st.close()


@pytest.mark.parametrize("integ,per,block,n_it,lanes", [
    ("euler", 4.5, 256, 1000, (4, 16)), ("euler_fma", 4.5, 128, 1000, (1, 16)), ("rk4", 4.5, 100, 640, (4, 16))])
def test_mix_without_room_and_captured(lz, simds, integ, per, block, n_it, lanes):
    import torch

    prm = dict(n_it=n_it, block_len=block, integrator=integ)
    chains = int(per * simds)
    assert mix_of(lz, simds, prm, chains) == lanes
    P = np.random.default_rng(chains).integers(0, 256, chains * block - 3, dtype=np.uint8)
    want = oracle.encrypt(b"plan", P, nthreads=ORACLE_THREADS, **prm)
    dP = to_dev(P)
    big_ctx, ctx = lz.Context(0), lz.Context(0, lz.params(**prm))
    big = torch.zeros(simds * 64 * 256, dtype=torch.uint8, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    big_ctx.encrypt(big, b"big", stream=s1)  # a wave on every SIMD, for longer than the three
    outs = [ctx.encrypt(dP, b"plan", stream=s2) for _ in range(3)]
    for k, o in enumerate(outs):
        assert np.array_equal(host(o), want), k
    C = torch.zeros(len(P) + 24, dtype=torch.uint8, device="cuda")
    new = lz.Context(0, lz.params(**prm))
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        new.encrypt(dP, b"plan", out=C)
    for k in range(3):
        C.zero_()
        g.replay()
        assert np.array_equal(host(C), want), k
        assert np.array_equal(host(ctx.encrypt(dP, b"plan")), want), k


def batch_case(lz, prm, lens, seed):
    """A batch of messages of these lengths, replayed, against the oracle; and decrypted."""
    import torch

    rng = np.random.default_rng(seed)
    pws = [b"m%d" % (i % 7) for i in range(len(lens))]
    data = rng.integers(0, 256, sum(lens), dtype=np.uint8)
    in_off, out_off = np.concatenate([[0], np.cumsum(lens)[:-1]]), lz.packed_offsets(lens, 24)
    ctx = lz.Context(0, lz.params(**prm))
    out = torch.zeros(out_off[1], dtype=torch.uint8, device="cuda")
    b = lz.Batch(ctx, False, lens, pws, to_dev(data), in_off, out, out_off[0])
    for replay in range(3):
        out.zero_()
        b.encrypt()
        got = host(out)
        if replay == 0:
            first = got
            for i in sorted({*range(min(120, len(lens))), *range(max(0, len(lens) - 120), len(lens))}):
                n = lens[i]
                want = oracle.encrypt(pws[i], data[in_off[i]:in_off[i] + n], nthreads=ORACLE_THREADS if n > 4096 else 1, **prm)
                o = int(out_off[0][i])
                assert np.array_equal(got[o:o + n + 24], want), (i, n)
        assert np.array_equal(got, first), replay
    plain = torch.zeros(len(data), dtype=torch.uint8, device="cuda")
    st = torch.full((len(lens),), 99, dtype=torch.int32, device="cuda")
    d = lz.Batch(ctx, True, lens, pws, out, out_off[0], plain, in_off)
    d.decrypt(st)
    assert np.array_equal(host(plain), data) and not host(st).any()


def lengths(n_full, tails, block, seed):
    rng = np.random.default_rng(seed)
    whole = rng.multinomial(n_full, np.ones(tails) / tails)
    return [int(w) * block + int(t) for w, t in zip(whole, rng.integers(1, block, tails))] + [0]


@pytest.mark.parametrize("integ,per,tails,block,n_it,lanes", [
    ("euler", 4.5, 900, 128, 1000, (4, 16)), ("euler_fma", 4.5, 2000, 128, 1000, (1, 16)), ("rk4", 4.5, 9, 100, 640, (4, 16)),
    ("rk4", 18, 700, 61, 150, (1, 4)), ("euler", 20, 40, 1000, 300, (1, 4))])
def test_mix_batches(lz, simds, integ, per, tails, block, n_it, lanes):
    prm = dict(n_it=n_it, block_len=block, integrator=integ)
    n_full = int(per * simds) - tails
    assert n_full >= tails + 1 and mix_of(lz, simds, prm, n_full + tails + 1) == lanes
    say(integ, n_full, tails)
    batch_case(lz, prm, lengths(n_full, tails, block, tails), tails)


SEG = [("euler", 37, 300), ("euler", 30, 300), ("euler_fma", 30, 640), ("rk4", 37, 100)]


@pytest.mark.parametrize("integ,block,n_it", SEG)
@pytest.mark.parametrize("times,more", [(1, 1), (1, 1 / 3), (2, 7), (3, 1 / 2), (5, 1 / 2)])
def test_segment_messages(lz, simds, integ, block, n_it, times, more):
    prm = dict(n_it=n_it, block_len=block, integrator=integ)
    waves = times * simds + (more if isinstance(more, int) else int(more * simds))
    p = lz.unit_plan(lz.params(**prm), simds, waves * 64 - 5)
    assert p.seg_waves == simds + waves % simds and block % p.seg_len  # a shorter last segment
    say(integ, block, waves, p.segs, p.seg_len)
    rng = np.random.default_rng(waves)
    both_ways(lz, prm, rng.integers(0, 256, (waves * 64 - 5) * block - 3, dtype=np.uint8))


@pytest.mark.parametrize("integ,block,n_it", SEG)
@pytest.mark.parametrize("full,tails", [((1, 64 * 90), 700), ((1, -64), 640), ((3, 17), 5000)])
def test_segment_batches(lz, simds, integ, block, n_it, full, tails):
    prm = dict(n_it=n_it, block_len=block, integrator=integ)
    n_full = full[0] * simds * 64 + full[1]
    lens = lengths(n_full, tails, block, tails)
    # the longest chain of each of the last waves: whole blocks first, then the partial ones, the longest first
    last = sorted((n % block for n in lens), reverse=True)
    chains = n_full + len(last)
    waves = (chains + 63) // 64
    g = (waves - (simds + waves % simds) + np.arange(simds + waves % simds)) * 64
    p = lz.unit_plan(lz.params(**prm), simds, chains, [block if x < n_full else last[x - n_full] for x in g])
    assert p.seg_waves == simds + waves % simds
    say(integ, block, waves, p.segs, p.seg_len, list(p.seg_off[:p.segs + 1]))
    batch_case(lz, prm, lens, tails)


def test_batch_of_many_sequential_messages(lz, simds):
    """block_len 2^32 - 1, each message one chain, more than one wave per SIMD."""
    prm = dict(n_it=20, block_len=(1 << 32) - 1)
    lens = [int(n) for n in np.random.default_rng(1).integers(0, 40, simds * 64 + 3000)]
    batch_case(lz, prm, lens, 1)
