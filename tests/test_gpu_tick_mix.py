"""Server ticks between two lane layouts (some requests with a lane per chain and the rest with four, by different byte
counts): bursts of a quarter to all of one wave per SIMD, both directions, against the plain path, which the
oracle pins."""
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


@pytest.mark.parametrize("integ", ["euler", "rk4", "euler_fma"])
@pytest.mark.parametrize("part,tick,biggest", [(0.27, 16, 300), (0.4, 7, 2000), (0.6, 1, 40), (0.9, 33, 700), (0.5, 16, 20000)])
def test_bursts(lz, integ, part, tick, biggest):
    import torch

    B = 64
    rng = np.random.default_rng(tick + biggest)
    wave = 4 * torch.cuda.get_device_properties(0).multi_processor_count * 64
    ctx = lz.Context(0, lz.params(n_it=20, block_len=B, integrator=integ))
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
    say(integ, part, tick, len(sizes), chains)
    srv = lz.Server(ctx, hbm_budget=1 << 30, tick_bytes=tick)
    for burst in range(2):
        for d in dst:
            d.zero_()
        torch.cuda.synchronize()
        at = lz.now_ns()
        srv.submit_many(list(range(len(sizes))), dec, pws, [s.data_ptr() for s in src], sizes, [d.data_ptr() for d in dst],
                        [at] * len(sizes))
        status, end = {}, time.monotonic() + 60
        while len(status) < len(sizes) and time.monotonic() < end:
            for rid, st, *_ in srv.poll(4096, 100):
                status[rid] = st
        assert status == {i: 0 for i in range(len(sizes))}
        for i, d in enumerate(dst):
            assert torch.equal(d, P[i] if dec[i] else C[i]), (burst, i, sizes[i])
    bytes_done = srv.stats()["chain_bytes"]
    srv.close()
    assert bytes_done == 2 * sum(sizes)
