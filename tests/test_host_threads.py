"""The host conversions' threads: calls at the same time, after the threads were ended, and in a forked child."""
import multiprocessing
import os
import subprocess
import sys
import threading
import time

import numpy as np
import pytest

from paper_1805_10692_amd import binding as B
from test_prepare_errors import HERE, fake  # noqa: F401  (a HIP runtime without a device that counts the threads a thread starts)


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


def test_threads_sleep_after_a_call_that_stands_alone():
    """What the process spends when the call has returned: a thread that polls for 250 us shows, the few dozen us before it sleeps do not."""
    others = min(len(os.sched_getaffinity(0)), 16) - 1
    if others < 1:
        pytest.skip("one processor")
    rng = np.random.default_rng(5)
    cb = np.array([0.0, 1.0, 2.0], np.float32)
    W = rng.choice(cb, size=(1024, 600)).astype(np.float32)
    spent = []
    for _ in range(32):
        time.sleep(0.02)
        h = B.cer_encode(W, cb)
        t = time.process_time()
        time.sleep(0.005)
        spent.append(time.process_time() - t)
        B.cer_free(h)
    # (polling: 1 to 2.2 ms with seven threads; without 0.03 to 1, the lowest quarter up to 0.3)
    assert sorted(spent)[8] < 100e-6 * others


BUSY = """
import ctypes, threading
import numpy as np
from paper_1805_10692_amd import binding as B
fake = ctypes.CDLL(None)
rng = np.random.default_rng(0)
cb = np.array([0.0, 1.0, 2.0], np.float32)
large, W = (rng.choice(cb, size=s, p=[0.4, 0.3, 0.3]).astype(np.float32) for s in ((2048, 4096), (512, 600)))
B.cer_free(B.cer_encode(large, cb))  # the waiting threads are there
stop = threading.Event()

def others():
    while not stop.is_set():
        B.cer_free(B.cer_encode(large, cb))

t = threading.Thread(target=others)
t.start()
started, out = [], np.empty_like(W)
for _ in range(60):
    a = fake.fake_hip_threads()
    h = B.cer_encode(W, cb)
    b = fake.fake_hip_threads()
    assert np.array_equal(B.cer_decode(h), W)
    started += [b - a, fake.fake_hip_threads() - b]
    B.cer_free(h)
stop.set()
t.join()
print(max(started))
"""


ALONE = """
import ctypes, os
import numpy as np
from paper_1805_10692_amd import binding as B
fake = ctypes.CDLL(None)
cb = np.array([0.0, 1.0, 2.0], np.float32)
W = np.random.default_rng(0).choice(cb, size=(SHAPE)).astype(np.float32)
before = fake.fake_hip_threads()
h = B.cer_encode(W, cb)
assert np.array_equal(B.cer_decode(h), W)
print(fake.fake_hip_threads() - before)
"""


@pytest.mark.parametrize("m,n", [(16, 1000), (300, 900), (1100, 1200)])
def test_processors_are_left_to_others(fake, m, n):  # noqa: F811
    """A thread per 16 Ki elements on three quarters of the processors, on more only where there is one for every 64 Ki."""
    processors = len(os.sched_getaffinity(0))
    work = m * n
    few, more = min(16, processors, m, -(-work // 65536)), min(16, processors * 3 // 4, m, -(-work // 16384))
    env = dict(os.environ, LD_PRELOAD=fake, PYTHONPATH=os.path.dirname(HERE))
    out = subprocess.run([sys.executable, "-c", ALONE.replace("SHAPE", f"{m}, {n}")], env=env, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert int(out.stdout) == max(1, few, more) - 1


def test_few_threads_are_started_where_the_waiting_ones_are_busy(fake):  # noqa: F811
    """Starting a thread takes some 10 us: one for every 64 Ki elements beside another conversion, none for the copy of the arrays (400 KB)."""
    if len(os.sched_getaffinity(0)) < 8:
        pytest.skip("as many processors as threads")
    env = dict(os.environ, LD_PRELOAD=fake, PYTHONPATH=os.path.dirname(HERE))
    out = subprocess.run([sys.executable, "-c", BUSY], env=env, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert 0 < int(out.stdout) <= (512 * 600 + 65535) // 65536 - 1


@pytest.mark.parametrize("values", [1, 2, 3, 17, 200])
@pytest.mark.parametrize("m,n", [(1, 16384), (2, 8193), (16, 1025), (33, 16385), (301, 1091)])
def test_shares_of_the_threads(m, n, values):
    """Around the sizes from which another thread helps; counters of few and of many values."""
    rng = np.random.default_rng(m * 1000 + values)
    cb = ((np.arange(values) - values // 2) * 0.5).astype(np.float32)
    W = cb[np.minimum(rng.geometric(0.4, size=(m, n)) - 1, values - 1)]
    for encode, decode in ((B.cer_encode, B.cer_decode), (B.cser_encode, B.cser_decode)):
        h = encode(W, cb)
        assert np.array_equal(decode(h), W)
        count = B.cer_get_array(h, B.CER_ARRAY_COUNT)
        assert np.array_equal(count, np.sort(np.unique(W, return_counts=True)[1])[::-1])
        B.cer_free(h)


@pytest.mark.gpu
@pytest.mark.parametrize("indexed", [131071, 131072, 131073, 131103, 400001])
def test_arrays_on_their_way_to_the_device(indexed):
    """Index arrays around the size from which threads share the copy, in whole and in odd shares."""
    import torch
    m, n = 512, 1024
    cb = np.array([0.0, 1.0, -2.0], np.float32)
    W = np.zeros(m * n, np.float32)
    at = np.random.default_rng(indexed).permutation(m * n)[:indexed]
    W[at] = np.where(at % 3 == 0, np.float32(1.0), np.float32(-2.0))
    W = W.reshape(m, n)
    if indexed > m * n // 2:
        W = np.where(W == 0, np.float32(5.0), W)
        cb = np.array([5.0, 1.0, -2.0], np.float32)
    h = B.cer_encode(W, cb)
    out = torch.empty((m, n), dtype=torch.float32, device="cuda")
    B.cer_decode_device(h, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), W)
    B.cer_free(h)
