"""The launch plans on the host (no GPU): every block length that the parameters take, up to the sequential
version's 2^32 - 1; and each plan run through here, task by task, against what the kernels assume of it."""
import ctypes

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
