"""Server ticks between two lane layouts at step counts where they pay, and not where a tick is too short to: bursts of requests of
all kinds against the plain path, with the tick count as the witness (a mixed tick gives most chains fewer bytes)."""
import time

import numpy as np
import pytest

from gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

@pytest.fixture(scope="module")
def lz():
    need_gpu()
    import paper_1201_3114_amd as lz

    return lz


def run_burst(lz, integ, n_it, B, part, tick, biggest):
    """A burst of `part` of a wave per SIMD, half of it decryptions; the ticks it took."""
    import torch

    rng = np.random.default_rng(tick + biggest)
    wave = 4 * torch.cuda.get_device_properties(0).multi_processor_count * 64
    ctx = lz.Context(0, lz.params(n_it=n_it, block_len=B, integrator=integ))
    sizes, chains = [0, 1, B, B + 1], 5
    while chains < part * wave:
        nb = int(rng.integers(1, min(biggest, int(part * wave) - chains + 1) + 1))
        sizes.append(nb * B - int(rng.integers(0, B)))
        chains += nb
    pws = [b"tick %d" % (i % 5) for i in range(len(sizes))]
    P = [torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda") for n in sizes]
    C = [ctx.encrypt(p, pw) for p, pw in zip(P, pws)]
    dec = [i % 2 == 1 for i in range(len(sizes))]
    dst = [torch.zeros(n + (0 if d else 24), dtype=torch.uint8, device="cuda") for n, d in zip(sizes, dec)]
    src = [c if d else p for p, c, d in zip(P, C, dec)]
    torch.cuda.synchronize()
    say(integ, n_it, part, tick, len(sizes), chains)
    srv = lz.Server(ctx, hbm_budget=1 << 30, tick_bytes=tick)
    at = lz.now_ns()
    srv.submit_many(list(range(len(sizes))), dec, pws, [s.data_ptr() for s in src], sizes, [d.data_ptr() for d in dst],
                    [at] * len(sizes))
    status, end = {}, time.monotonic() + 60
    while len(status) < len(sizes) and time.monotonic() < end:
        for rid, st, *_ in srv.poll(4096, 20):
            status[rid] = st
    assert status == {i: 0 for i in range(len(sizes))}
    for i, d in enumerate(dst):
        assert torch.equal(d, P[i] if dec[i] else C[i]), (i, sizes[i])
    stats = srv.stats()
    srv.close()
    assert stats["chain_bytes"] == sum(sizes)
    return stats["ticks"]


@pytest.mark.parametrize("integ,n_it", [("euler", 3000), ("rk4", 600)])
@pytest.mark.parametrize("part,tick,biggest", [(0.27, 16, 300), (0.4, 11, 2000), (0.6, 33, 400), (0.5, 16, 20000)])
def test_mixed(lz, integ, n_it, part, tick, biggest):
    ticks = run_burst(lz, integ, n_it, 64, part, tick, biggest)
    say("ticks", ticks)
    assert ticks > -(-64 // tick)


@pytest.mark.parametrize("part,tick,biggest", [(0.27, 16, 300), (0.5, 16, 20000)])
def test_short_ticks_are_not_mixed(lz, part, tick, biggest):
    ticks = run_burst(lz, "euler", 10, 256, part, tick, biggest)
    say("ticks", ticks)
    # the first tick may come before the last request; mixed ticks would be 18 or more
    assert ticks <= 256 // tick + 1
