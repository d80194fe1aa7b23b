"""Products that need temporaries, on several streams and from several threads: the blocks the library keeps between calls
never serve two products at once, whichever stream or thread returns them."""
import threading

import numpy as np
import pytest

import oracle
from paper_1805_10692_amd import binding as B
from paper_1805_10692_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [1, 3])
def test_streams_and_threads_share_the_kept_blocks(threads):
    dev = torch.device("cuda:0")
    w = wl.conv3x3(L=96, nonzero_dominant=True, scale=4)   # column sums, and a decoded matrix or strips' partial sums
    want = oracle.dot(oracle.encode(w.W, w.codebook, "cer"), w.X, threads=8)
    bound = 1e-5 * oracle.abs_dot_dense(w.W, w.X, threads=8)
    h = B.cer_encode(w.W, w.codebook)
    B.cer_prepare_strips(h)
    X = torch.from_numpy(w.X).to(dev)
    scales = [1.0, 2.0, 4.0, 8.0]                          # powers of two: the same rounding, another result
    Xs = [X * s for s in scales]
    torch.cuda.synchronize()
    bad = []

    def work():
        streams = [None, torch.cuda.Stream(), torch.cuda.Stream()]
        for path in (B.CER_PATH_STRIP, B.CER_PATH_DENSE):
            outs = []
            for i in range(24):
                Y = torch.empty((w.m, w.L), device=dev)
                torch.cuda.current_stream().synchronize()
                B.cer_matmul_ex(h, Xs[i % 4], Y, w.L, streams[i % 3], B.MatmulOpts(path=path))
                outs.append(Y)
            del streams[2]                                 # a stream that is gone while its blocks are kept
            torch.cuda.synchronize()
            streams.append(torch.cuda.Stream())
            for i, Y in enumerate(outs):
                err = np.abs(Y.cpu().numpy().astype(np.float64) / scales[i % 4] - want)
                if not (err <= bound).all():
                    bad.append((path, i))

    pool = [threading.Thread(target=work) for _ in range(threads)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    B.cer_trim()
    assert not bad, bad
    B.cer_free(h)


@pytest.mark.parametrize("side_stream", [False, True])
def test_a_freed_handles_memory_serves_the_next_one_in_order(side_stream):
    """A handle is freed while its products are still queued; the next handle of the same size, encoded on the null stream,
    takes over its device memory: every product shows its own matrix."""
    dev = torch.device("cuda:0")
    cb = np.array([-1.0, 0.0, 1.0, 2.0], np.float32)
    rng = np.random.default_rng(3)
    Ws = [rng.choice(cb, size=(700, 900), p=[0.1, 0.7, 0.1, 0.1]).astype(np.float32) for _ in range(4)]
    X = torch.from_numpy(rng.standard_normal((900, 40)).astype(np.float32)).to(dev)
    Wd = [torch.from_numpy(W).to(dev) for W in Ws]
    stream = torch.cuda.Stream() if side_stream else None
    torch.cuda.synchronize()
    outs = []
    for W in Wd:
        h = B.cer_encode_device(W, 700, 900, cb, "cer")
        for _ in range(20):
            Y = torch.empty((700, 40), device=dev)
            B.cer_matmul(h, X, Y, 40, stream)
        outs.append(Y)
        B.cer_free(h)
    torch.cuda.synchronize()
    for W, Y in zip(Ws, outs):
        want = W.astype(np.float64) @ X.cpu().numpy().astype(np.float64)
        bound = 1e-5 * (np.abs(W).astype(np.float64) @ np.abs(X.cpu().numpy()).astype(np.float64))
        assert (np.abs(Y.cpu().numpy() - want) <= bound).all()


def test_freeing_a_handle_does_not_wait_for_another_threads_encoder():
    """An encoder that takes over the memory of a handle with work still queued on a side stream waits for the device; a handle
    that is freed by another thread in the meantime is not held up by that."""
    dev = torch.device("cuda:0")
    cb = np.array([-1.0, 0.0, 1.0, 2.0], np.float32)
    rng = np.random.default_rng(5)
    W = rng.choice(cb, size=(700, 900), p=[0.1, 0.7, 0.1, 0.1]).astype(np.float32)
    other = B.cer_encode(rng.choice(cb, size=(2000, 1500)).astype(np.float32), cb)
    x1, y1 = torch.randn((900, 1), device=dev), torch.empty((700, 1), device=dev)
    big, xb, yb = (torch.randn((4096, 4096), device=dev) for _ in range(3))
    stream, done = torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    B.cer_trim()                                           # no other block of that size
    first = B.cer_encode(W, cb)
    B.cer_matmul(first, x1, y1, 1, stream)
    for _ in range(600):                                   # about a second on the side stream
        B.dense_matmul(big, xb, yb, 4096, 4096, 4096, stream)
    done.record(stream)
    B.cer_free(first)
    taken = []
    encoder = threading.Thread(target=lambda: taken.append(B.cer_encode(W, cb)))
    encoder.start()
    encoder.join(0.1)
    waiting = encoder.is_alive()                           # it is in its wait for the device
    B.cer_free(other)
    pending = not done.query()
    encoder.join()
    torch.cuda.synchronize()
    assert waiting and pending
    Y = torch.empty((700, 1), device=dev)
    B.cer_matmul(taken[0], x1, Y, 1)
    assert torch.equal(Y, y1)
    B.cer_free(taken[0])
    B.cer_trim()


def test_more_streams_than_kept_blocks():
    """Forty streams with work queued in front of their products hold forty temporaries at once, more than the list keeps: the
    oldest go back to the runtime while later ones are in use."""
    dev = torch.device("cuda:0")
    cb = np.array([0.0, 1.0, -0.75, 3.0], np.float32)
    rng = np.random.default_rng(9)
    W = rng.choice(cb, size=(300, 500), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
    X = rng.standard_normal((500, 70)).astype(np.float32)
    want = W.astype(np.float64) @ X.astype(np.float64)
    bound = 1e-5 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64))
    h = B.cer_encode(W, cb)
    Xd = torch.from_numpy(X).to(dev)
    big, xb, yb = (torch.randn((2048, 2048), device=dev) for _ in range(3))
    streams = [torch.cuda.Stream() for _ in range(40)]
    outs = [torch.full((300, 70), float("nan"), device=dev) for _ in streams]
    torch.cuda.synchronize()
    B.cer_trim()
    for _ in range(3):
        for s, Y in zip(streams, outs):
            B.dense_matmul(big, xb, yb, 2048, 2048, 2048, s)
            B.cer_matmul_ex(h, Xd, Y, 70, s, B.MatmulOpts(path=B.CER_PATH_DENSE))
    torch.cuda.synchronize()
    for Y in outs:
        assert (np.abs(Y.cpu().numpy() - want) <= bound).all()
    B.cer_trim()
    B.cer_free(h)
