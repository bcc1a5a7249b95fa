"""Messages and batches whose last waves run by a segment plan (chains cut in time, advanced in rounds),
against the oracle bit for bit: wave counts just past one, two and five waves per SIMD and just
below the next, ragged last blocks, tails of all lengths, every integrator, both directions."""
import numpy as np
import pytest

import oracle
from gpu_util import ORACLE_THREADS, host, need_gpu, say, to_dev

pytestmark = pytest.mark.gpu

B, N_IT = 16, 300  # steps enough that a plan's rounds pay (13 bytes: a length the segments do not divide)


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def simds():
    import torch

    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("integ,block", [("euler", B), ("euler", 13), ("euler_fma", B), ("rk4", B)])
@pytest.mark.parametrize("waves", ["S+1", "S+S//3", "2S-1", "2S+7", "5S+S//2"])
def test_plain(lz, integ, block, waves):
    if integ == "rk4" and waves[0] in "25":
        pytest.skip("the oracle's time")
    S = simds()
    W = eval(waves.replace("2S", "2*S").replace("5S", "5*S"), {"S": S})
    rng = np.random.default_rng(W)
    n = (W * 64 - 5) * block - 3  # a last wave of 59 chains, the last of them short
    P = rng.integers(0, 256, n, dtype=np.uint8)
    ctx = lz.Context(0, lz.params(n_it=N_IT, block_len=block, integrator=integ))
    say(integ, block, W, n)
    C = ctx.encrypt(to_dev(P), b"segments")
    want = oracle.encrypt(b"segments", P, nthreads=ORACLE_THREADS, n_it=N_IT, block_len=block, integrator=integ)
    assert np.array_equal(host(C), want)
    assert np.array_equal(host(ctx.decrypt(C, b"segments")), P)
    bad = C.clone()
    bad[n // 2] ^= 1
    with pytest.raises(lz.IntegrityError):
        ctx.decrypt(bad, b"segments")


@pytest.mark.parametrize("integ", ["euler", "euler_fma"])
@pytest.mark.parametrize("full,tails", [("S*64+64*90", 700), ("S*64-64*3", 640), ("3*S*64+17", 5000)])
def test_batch(lz, integ, full, tails):
    """`tails` messages of which each ends in a partial block, `full` whole blocks among them; an empty message."""
    import torch

    S = simds()
    rng = np.random.default_rng(tails)
    n_full = eval(full, {"S": S})
    whole = rng.multinomial(n_full, np.ones(tails) / tails)
    lens = [int(w) * B + int(t) for w, t in zip(whole, rng.integers(1, B, tails))] + [0]
    pws = [b"m%d" % i for i in range(len(lens))]
    data = rng.integers(0, 256, sum(lens), dtype=np.uint8)
    in_off, out_off = np.concatenate([[0], np.cumsum(lens)[:-1]]), lz.packed_offsets(lens, 24)
    out = torch.zeros(out_off[1], dtype=torch.uint8, device="cuda")
    ctx = lz.Context(0, lz.params(n_it=N_IT, block_len=B, integrator=integ))
    say(integ, n_full, tails)
    b = lz.Batch(ctx, False, lens, pws, to_dev(data), in_off, out, out_off[0])
    for replay in range(3):
        out.zero_()
        b.encrypt()
        got = host(out)
        if replay == 0:
            first = got
            for i, n in enumerate(lens):
                want = oracle.encrypt(pws[i], data[in_off[i]:in_off[i] + n], nthreads=ORACLE_THREADS if n > 4096 else 1,
                                      n_it=N_IT, block_len=B, integrator=integ)
                o = int(out_off[0][i])
                assert np.array_equal(got[o:o + n + 24], want), (integ, i, n)
        assert np.array_equal(got, first), replay
    plain = torch.zeros(len(data), dtype=torch.uint8, device="cuda")
    st = torch.full((len(lens),), 99, dtype=torch.int32, device="cuda")
    d = lz.Batch(ctx, True, lens, pws, out, out_off[0], plain, in_off)
    d.decrypt(st)
    assert np.array_equal(host(plain), data) and not host(st).any()


def test_captured(lz):
    """The first call of a context, with a segment plan, inside a graph: replayed three times with eager work between."""
    import torch

    S = simds()
    rng = np.random.default_rng(3)
    P = rng.integers(0, 256, (S + S // 4) * 64 * B - 5, dtype=np.uint8)
    ctx = lz.Context(0, lz.params(n_it=N_IT, block_len=B))
    dP = to_dev(P)
    C = torch.zeros(len(P) + 24, dtype=torch.uint8, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        ctx.encrypt(dP, b"captured", out=C)
    want = oracle.encrypt(b"captured", P, nthreads=ORACLE_THREADS, n_it=N_IT, block_len=B)
    for k in range(3):
        C.zero_()
        g.replay()
        assert np.array_equal(host(C), want), k
        assert np.array_equal(host(lz.Context(0, lz.params(n_it=N_IT, block_len=B)).encrypt(dP, b"captured")), want), k
