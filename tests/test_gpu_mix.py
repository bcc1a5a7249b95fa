"""Messages and stream updates that run by a mix plan (rounds in which some chains take one layout and the rest
the next wider one), against the oracle bit for bit: chain counts from just above one layout's
limit to just below the next, ragged ends, head and tail blocks of updates, and no room on the device."""
import numpy as np
import pytest

import oracle
from gpu_util import ORACLE_THREADS, host, need_gpu, say, to_dev

pytestmark = pytest.mark.gpu

B = 64
N_IT = {"euler": 600, "euler_fma": 900, "rk4": 150}  # enough that the rounds pay


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def simds():
    import torch

    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


# chains per SIMD, and a few more: between 16 and 64 the layouts of 1 and 4 lanes meet (1 and 16 lanes for the fused
# map, from 4), between 4 and 16 those of 4 and 16
CASES = [("euler", 16, 5), ("euler", 24, 0), ("euler", 41, 33), ("euler", 60, -1), ("euler", 4, 3), ("euler", 6, -2),
         ("euler", 9, 7), ("euler_fma", 4, 9), ("euler_fma", 7, 1), ("euler_fma", 20, 0), ("rk4", 17, 3), ("rk4", 30, -7),
         ("rk4", 4, 5), ("rk4", 7, -1)]


@pytest.mark.parametrize("integ,per,more", CASES)
def test_plain(lz, integ, per, more):
    rng = np.random.default_rng(per)
    nb = per * simds() + more
    n = nb * B - 11
    prm = dict(n_it=N_IT[integ], block_len=B, integrator=integ)
    ctx = lz.Context(0, lz.params(**prm))
    P = rng.integers(0, 256, n, dtype=np.uint8)
    say(integ, nb, n)
    C = ctx.encrypt(to_dev(P), b"mix")
    want = oracle.encrypt(b"mix", P, nthreads=ORACLE_THREADS, **prm)
    assert np.array_equal(host(C), want)
    assert np.array_equal(host(ctx.decrypt(C, b"mix")), P)
    bad = C.clone()
    bad[n + 3] ^= 1
    with pytest.raises(lz.IntegrityError):
        ctx.decrypt(bad, b"mix")


@pytest.mark.parametrize("integ,per", [("euler", 20), ("euler", 5), ("euler_fma", 5)])
def test_stream_updates(lz, integ, per):
    """Updates whose first block is half done and whose last is left half done; a short one between."""
    rng = np.random.default_rng(per + 100)
    prm = dict(n_it=N_IT[integ], block_len=B, integrator=integ)
    ctx = lz.Context(0, lz.params(**prm))
    cuts = [0, per * simds() * B + 13, per * simds() * B + 40, 2 * per * simds() * B + 64 + 50]
    P = rng.integers(0, 256, cuts[-1], dtype=np.uint8)
    want = oracle.encrypt(b"mix", P, nthreads=ORACLE_THREADS, **prm)
    for decrypt in (False, True):
        src = to_dev(want[:len(P)] if decrypt else P)
        st = lz.Stream(ctx, decrypt, b"mix")
        out = [st.update(src[a:e].clone()) for a, e in zip(cuts, cuts[1:])]
        body = np.concatenate([host(o) for o in out])
        if decrypt:
            assert np.array_equal(body, P), integ
            st.finish(to_dev(want[len(P):]))  # raises if the tag differs
        else:
            assert np.array_equal(np.concatenate([body, host(st.finish())]), want), integ
        st.close()


@pytest.mark.parametrize("integ,per", [("euler", 20), ("euler", 6)])
def test_no_room_and_capture(lz, integ, per):
    import torch

    rng = np.random.default_rng(per + 200)
    prm = dict(n_it=N_IT[integ], block_len=B, integrator=integ)
    big_ctx, ctx = lz.Context(0, lz.params(**prm)), lz.Context(0, lz.params(**prm))
    big = torch.randint(0, 256, (4 * simds() * 64 * B,), dtype=torch.uint8, device="cuda")
    P = rng.integers(0, 256, per * simds() * B - 3, dtype=np.uint8)
    want = oracle.encrypt(b"mix", P, nthreads=ORACLE_THREADS, **prm)
    dP = to_dev(P)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    C0 = big_ctx.encrypt(big, b"big", stream=s1)
    outs = [ctx.encrypt(dP, b"mix", stream=s2) for _ in range(3)]
    torch.cuda.synchronize()
    for k, o in enumerate(outs):
        assert np.array_equal(host(o), want), k
    assert torch.equal(big_ctx.decrypt(C0, b"big"), big)
    new = lz.Context(0, lz.params(**prm))
    C = torch.zeros(len(P) + 24, dtype=torch.uint8, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        new.encrypt(dP, b"mix", out=C)
    for k in range(3):
        C.zero_()
        g.replay()
        assert np.array_equal(host(C), want), k
        assert np.array_equal(host(ctx.encrypt(dP, b"mix")), want), k


@pytest.mark.parametrize("per,block", [(5, 4096), (20, 1000), (4, 300)])
def test_long_blocks(lz, per, block):
    """Rounds of more bytes, as many as of a default block."""
    rng = np.random.default_rng(block)
    n = (per * simds() + 3) * block - 77
    prm = dict(n_it=40, block_len=block)
    ctx = lz.Context(0, lz.params(**prm))
    P = rng.integers(0, 256, n, dtype=np.uint8)
    C = ctx.encrypt(to_dev(P), b"mix")
    assert np.array_equal(host(C), oracle.encrypt(b"mix", P, nthreads=ORACLE_THREADS, **prm))
    assert np.array_equal(host(ctx.decrypt(C, b"mix")), P)


@pytest.mark.parametrize("integ,per,tails", [("euler", 20, 40), ("euler", 33, 5000), ("euler", 5, 9), ("euler_fma", 6, 700),
                                             ("rk4", 18, 100), ("euler", 6, 3072)])
@pytest.mark.parametrize("room", [True, False])
def test_batch(lz, integ, per, tails, room):
    """Messages with partial last blocks and an empty one; replays, also beside work that leaves no room."""
    import torch

    rng = np.random.default_rng(per + tails)
    n_full = per * simds() - tails
    whole = rng.multinomial(n_full, np.ones(tails) / tails)
    lens = [int(w) * B + int(t) for w, t in zip(whole, rng.integers(1, B, tails))] + [0]
    pws = [b"m%d" % (i % 7) for i in range(len(lens))]
    data = rng.integers(0, 256, sum(lens), dtype=np.uint8)
    in_off, out_off = np.concatenate([[0], np.cumsum(lens)[:-1]]), lz.packed_offsets(lens, 24)
    prm = dict(n_it=N_IT[integ], block_len=B, integrator=integ)
    ctx = lz.Context(0, lz.params(**prm))
    big = torch.zeros((4 * simds() * 64 * B,), dtype=torch.uint8, device="cuda")
    out = torch.zeros(out_off[1], dtype=torch.uint8, device="cuda")
    say(integ, n_full, tails, room)
    b = lz.Batch(ctx, False, lens, pws, to_dev(data), in_off, out, out_off[0])
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for replay in range(3):
        out.zero_()
        torch.cuda.synchronize()
        if not room:
            lz.Context(0, lz.params(**prm)).encrypt(big, b"big", stream=s1)
        b.encrypt(stream=s2)
        torch.cuda.synchronize()
        got = host(out)
        if replay == 0:
            first = got
            for i in sorted({*range(min(300, len(lens))), *range(max(0, len(lens) - 300), len(lens))}):
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
