"""entropy() on two threads and two streams of one context: a call waits for the work ahead of it on its own stream, not
for the other call's."""
import threading
import time

import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev

pytestmark = pytest.mark.gpu


def test_a_call_does_not_wait_for_another_streams_work():
    need_gpu()
    import torch

    import paper_1201_3114_amd as lz

    ctx, slow_ctx = lz.Context(0), lz.Context(0, lz.params(block_len=4096))
    hist = lz.histogram(ctx, to_dev(np.arange(4096) % 256))
    slow = to_dev(np.zeros(4096, np.uint8))  # one chain of 4096 bytes: some 200 ms on one wave
    out = torch.empty(4096 + 24, dtype=torch.uint8, device="cuda")
    assert lz.entropy(ctx, hist) == 8.0
    s1 = torch.cuda.Stream()
    took = []
    for _ in range(8):  # until a stream whose hardware queue is not s1's
        s2 = torch.cuda.Stream()
        lz.entropy(ctx, hist, stream=s2)
        torch.cuda.synchronize()
        slow_ctx.encrypt(slow, b"slow", out=out, stream=s1)
        ends = {}

        def first():
            assert lz.entropy(ctx, hist, stream=s1) == 8.0
            ends["first"] = time.monotonic()

        t = threading.Thread(target=first)
        start = time.monotonic()
        t.start()
        time.sleep(0.02)
        assert lz.entropy(ctx, hist, stream=s2) == 8.0
        ends["second"] = time.monotonic()
        t.join()
        took.append((ends["first"] - start, ends["second"] - start))
        if took[-1][1] < 0.5 * took[-1][0]:
            break
    say(took)
    assert took[-1][0] > 0.1 and took[-1][1] < 0.5 * took[-1][0]


def test_more_threads_than_words():
    need_gpu()
    import torch

    import paper_1201_3114_amd as lz

    ctx = lz.Context(0)
    data = [np.arange(5000 + i) % (2 + i) for i in range(96)]
    hists = [lz.histogram(ctx, to_dev(d % 256)) for d in data]
    want = [lz.entropy(ctx, h) for h in hists]
    torch.cuda.synchronize()
    got = [None] * 96

    def work(i):
        got[i] = [lz.entropy(ctx, hists[i]) for _ in range(10)]

    threads = [threading.Thread(target=work, args=(i,)) for i in range(96)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [[w] * 10 for w in want]
