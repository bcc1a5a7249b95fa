"""The launch plans on the host (no GPU): every block length that the parameters take, up to the sequential
version's 2^32 - 1; and each plan run through here, task by task, against what the kernels assume of it."""

import numpy as np
import pytest

import paper_1201_3114_amd as lz

SIMDS = 1024
INTEG = ["euler", "euler_fma", "rk4"]


@pytest.mark.parametrize("block", [1 << 20, (1 << 30) - 1, 1 << 31, (1 << 32) - 5, (1 << 32) - 1])
@pytest.mark.parametrize("chains", [100, 5000, 20000, 65536, 65537, 70000, 140000])
def test_sequential_block_lengths(block, chains):
    """Messages of 300 bytes as one chain each: more than one wave per SIMD too."""
    prm = lz.params(block_len=block)
    waves = (chains + 63) // 64
    p = lz.unit_plan(prm, SIMDS, chains, [300] * (SIMDS + waves % SIMDS))
    assert p.seg_waves == 0
    lz.unit_plan(prm, SIMDS, chains)


def check_mix(p, chains, block):
    ga, gb = p.mix_lanes
    la, lb = p.mix_bytes
    assert 0 < p.mix_first < p.mix_units and p.mix_unit == 64 // ga
    assert p.mix_units * p.mix_unit >= chains > (p.mix_units - 1) * p.mix_unit
    assert p.mix_first + (p.mix_units - p.mix_first) * (gb // ga) <= SIMDS  # waves of a round
    assert p.mix_units * p.mix_unit <= 2 * 64 * SIMDS  # checkpoints
    pos = np.zeros(p.mix_units, np.int64)
    turns = np.zeros(p.mix_units, np.int64)
    u = np.arange(p.mix_units)
    for r in range(p.mix_rounds):
        # a unit's turns in ga lanes before round r, from the round's number alone: the multiples u, u + units, ... below r first
        ra = r * p.mix_first
        assert np.array_equal(turns, np.where(ra > u, (ra - 1 - u) // p.mix_units + 1, 0))
        assert np.array_equal(pos, turns * la + (r - turns) * lb)
        first = (r * p.mix_first + np.arange(p.mix_first)) % p.mix_units
        assert len(set(first.tolist())) == p.mix_first
        pos += lb
        pos[first] += la - lb
        turns[first] += 1
    assert pos.min() >= block


def check_seg(p, chains, block, lens):
    waves = (chains + 63) // 64
    off = list(p.seg_off[:p.segs + 1])
    assert SIMDS <= p.seg_waves < 2 * SIMDS and (waves - p.seg_waves) % SIMDS == 0 and p.segs <= 32
    assert p.segs * p.seg_len >= block > (p.segs - 1) * p.seg_len
    assert off[0] == 0 and p.seg_rounds == -(-off[-1] // SIMDS)
    per = [b - a for a, b in zip(off, off[1:])]
    assert per[0] == p.seg_waves and all(a >= b for a, b in zip(per, per[1:]))
    last = {}  # wave -> the round of its latest task
    for t in range(off[-1]):
        s = next(i for i in range(p.segs) if t < off[i + 1])
        w, r = t - off[s], t // SIMDS
        assert last.get(w, -1) < r  # after its segment before, in a later round
        last[w] = r
    for w in range(p.seg_waves):  # every wave has the tasks of its longest chain
        need = -(-max(lens[w] if lens is not None else block, 1) // p.seg_len)
        assert sum(w < n for n in per) >= need


@pytest.mark.parametrize("integ", INTEG)
def test_plans_cover_every_byte_once(integ):
    rng = np.random.default_rng(INTEG.index(integ))
    seen = {"mix": 0, "seg": 0, "tails": 0}
    for _ in range(400):
        block = int(np.exp(rng.uniform(np.log(13), np.log(5000))))
        prm = lz.params(n_it=int(np.exp(rng.uniform(np.log(50), np.log(4000)))), block_len=block, integrator=integ)
        chains = int(np.exp(rng.uniform(np.log(4 * SIMDS), np.log(300 * SIMDS))))
        waves = (chains + 63) // 64
        n = SIMDS + waves % SIMDS
        lens = None
        if rng.random() < 0.5 and waves > SIMDS:  # partial blocks in the last waves
            lens = np.full(n, block)
            k = int(rng.integers(1, max(2, n - SIMDS + 1)))
            lens[n - k:] = np.sort(rng.integers(1, block + 1, k))[::-1]
        p = lz.unit_plan(prm, SIMDS, chains, lens)
        if p.mix_rounds:
            check_mix(p, chains, block)
            seen["mix"] += 1
        if p.seg_waves:
            check_seg(p, chains, block, lens)
            seen["seg"] += 1
            seen["tails"] += lens is not None
    assert min(seen.values()) >= 5, seen
