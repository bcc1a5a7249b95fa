"""Launches that spread a chain over several lanes (short messages, batches and stream updates), against the
oracle bit for bit: around the chain counts where the layout changes and the edges of a wave, with
step counts around the 60 and 120 steps of a loop iteration, and beside a launch that leaves no room for
the wide layout."""
import numpy as np
import pytest

import oracle
from gpu_util import ORACLE_THREADS, host, need_gpu, say, to_dev

pytestmark = pytest.mark.gpu

B = 6  # block length: short, so that the chain counts below stay small messages


@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def simds():
    import torch

    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


def edges():
    """Chain counts: a lane group, the waves of 4, 16 and 64 chains, one wave on every SIMD of each layout."""
    s = simds()
    return [1, 3, 4, 5, 16, 17, 63, 65, 4 * s, 4 * s + 1, 16 * s, 16 * s + 1]


@pytest.mark.parametrize("integ", ["euler", "euler_fma", "rk4"])
@pytest.mark.parametrize("n_it", [1, 59, 60, 119, 120, 241])
def test_plain_at_layout_edges(lz, integ, n_it):
    rng = np.random.default_rng(n_it)
    ctx = lz.Context(0, lz.params(n_it=n_it, block_len=B, integrator=integ))
    for nb in edges():
        n = nb * B - int(rng.integers(0, B))  # a ragged last block
        pw = b"lanes %d" % nb
        P = rng.integers(0, 256, n, dtype=np.uint8)
        say(integ, n_it, nb, n)
        C = ctx.encrypt(to_dev(P), pw)
        want = oracle.encrypt(pw, P, nthreads=ORACLE_THREADS, n_it=n_it, block_len=B, integrator=integ)
        assert np.array_equal(host(C), want), (integ, n_it, nb)
        assert np.array_equal(host(ctx.decrypt(C, pw)), P), (integ, n_it, nb)


@pytest.mark.parametrize("integ", ["euler", "euler_fma", "rk4"])
def test_batch_and_stream_at_layout_edges(lz, integ):
    import torch

    rng = np.random.default_rng(7)
    ctx = lz.Context(0, lz.params(n_it=61, block_len=B, integrator=integ))
    kw = dict(nthreads=ORACLE_THREADS, n_it=61, block_len=B, integrator=integ)
    for nb in edges():
        lens = [nb * B // 2 + 1, 0, nb * B - nb * B // 2 - 1]  # chains: about nb, an empty message among them
        pws = [b"a%d" % nb, b"b", b"c%d" % nb]
        data = rng.integers(0, 256, sum(lens), dtype=np.uint8)
        in_off = np.concatenate([[0], np.cumsum(lens)[:-1]])
        out_off, tot = lz.packed_offsets(lens, 24)
        out = torch.empty(tot, dtype=torch.uint8, device="cuda")
        say(integ, nb, lens)
        b = lz.Batch(ctx, False, lens, pws, to_dev(data) if len(data) else torch.empty(1, dtype=torch.uint8, device="cuda"),
                     in_off, out, out_off)
        b.encrypt()
        got = host(out)
        for i, n in enumerate(lens):
            want = oracle.encrypt(pws[i], data[in_off[i]:in_off[i] + n], **kw)
            assert np.array_equal(got[int(out_off[i]):int(out_off[i]) + n + 24], want), (integ, nb, i)
        b.close()
        # the same bytes as one message, cut inside blocks: head and tail chains beside whole blocks
        st = lz.Stream(ctx, False, b"s")
        cuts = sorted({0, 1, min(len(data), B + 2), len(data) // 2 + 1, len(data)})
        parts = [st.update(to_dev(data[a:e])) for a, e in zip(cuts, cuts[1:]) if e > a]
        tag = host(st.finish())
        body = np.concatenate([host(p) for p in parts]) if parts else data
        assert np.array_equal(np.concatenate([body, tag]), oracle.encrypt(b"s", data, **kw)), (integ, nb)


@pytest.mark.parametrize("integ", ["euler", "euler_fma", "rk4"])
def test_no_room_for_wide_launches(lz, integ):
    """Short messages queued while a message that fills the device runs: they may have to run with a chain
    per lane, and give the same bytes; afterwards, alone again, too."""
    import torch

    rng = np.random.default_rng(9)
    prm = dict(n_it=60, block_len=B, integrator=integ)
    big_ctx = lz.Context(0, lz.params(n_it=600, block_len=B, integrator=integ))
    big = torch.randint(0, 256, (8 * simds() * 64 * B,), dtype=torch.uint8, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = lz.Context(0, lz.params(**prm))
    P = rng.integers(0, 256, 16 * simds() * B - 3, dtype=np.uint8)
    want = oracle.encrypt(b"pw", P, nthreads=ORACLE_THREADS, **prm)
    dP = to_dev(P)
    torch.cuda.synchronize()
    C0 = big_ctx.encrypt(big, b"big", stream=s1)
    outs = [ctx.encrypt(dP, b"pw", stream=s2) for _ in range(4)]
    torch.cuda.synchronize()
    outs.append(ctx.encrypt(dP, b"pw"))
    for k, o in enumerate(outs):
        assert np.array_equal(host(o), want), (integ, k)
    assert torch.equal(big_ctx.decrypt(C0, b"big"), big)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 16383, 16384 + 5, 131072 + 31, (1 << 20) + 3])
def test_copies_of_unaligned_chunks(lz, n):
    """Deferred chunks: staged and copied out in pieces whose source and destination agree modulo 16 or not, of
    lengths around a move, a workgroup's turn and a piece; bytes beside them stay."""
    import torch

    rng = np.random.default_rng(n)
    ctx = lz.Context(0, lz.params(n_it=1, block_len=64))
    src = torch.from_numpy(rng.integers(0, 256, 3 * n + 64, dtype=np.uint8)).cuda()
    dst = torch.full((3 * n + 96,), 7, dtype=torch.uint8, device="cuda")
    at = [(5, 3), (5 + n, 3 + n + 8), (5 + 2 * n, 3 + 2 * n + 25)]  # (source, destination), gaps between the outputs
    st = lz.Stream(ctx, False, b"copies")
    for s, d in at:
        st.update_deferred(src[s:s + n], out=dst[d:d + n])
    tag = host(st.finish())
    want = oracle.encrypt(b"copies", host(src)[5:5 + 3 * n], nthreads=ORACLE_THREADS, n_it=1, block_len=64)
    got, keep = host(dst), np.full(3 * n + 96, 7, dtype=np.uint8)
    for i, (s, d) in enumerate(at):
        keep[d:d + n] = want[i * n:(i + 1) * n]
    assert np.array_equal(got, keep) and np.array_equal(tag, want[3 * n:])
