"""The host conversions' threads: calls at the same time, after the threads were ended, and in a forked child."""
import multiprocessing
import threading

import numpy as np
import pytest

from paper_1805_10692_amd import binding as B


def _round_trip(seed, m=300, n=1100):
    rng = np.random.default_rng(seed)
    cb = np.array([-1.5, 0.0, 0.25, 3.0, 7.0], np.float32)
    W = rng.choice(cb, size=(m, n), p=[0.1, 0.6, 0.1, 0.1, 0.1]).astype(np.float32)
    h = B.cer_encode(W, cb)
    ok = np.array_equal(B.cer_decode(h), W)
    B.cer_free(h)
    return ok


def test_calls_at_the_same_time():
    bad = []

    def work(i):
        for k in range(8):
            if not _round_trip(100 * i + k):
                bad.append((i, k))

    pool = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    assert not bad


def _child(q):
    q.put(_round_trip(7))


def test_after_a_fork():
    if B.lib().cer_last_hip_error() == 0:
        import torch
        if torch.cuda.is_available():
            pytest.skip("a process that has used the GPU is not forked")
    assert _round_trip(1)
    ctx = multiprocessing.get_context("fork")
    q = ctx.Queue()
    p = ctx.Process(target=_child, args=(q,))
    p.start()
    assert q.get(timeout=60)
    p.join(60)
    assert p.exitcode == 0


def test_threads_come_back_after_they_were_ended():
    assert _round_trip(2)
    try:
        B.cer_trim()                # without a GPU the rest of the call reports it
    except B.CerError:
        pass
    assert _round_trip(3)
