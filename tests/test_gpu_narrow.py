"""Batches of 2 to 8 columns by the library's own choice (csrc/cer_narrow.hip): every number of columns per pass, 8- and 16-bit
indices, one to four tiles of groups, rows shared by several waves, rows of several windows, unaligned X, non-zero Omega[0]."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(m, n, L, K, p0, zero, fmt, shift=0):
    """zero: position of 0 in the codebook (K // 2: 0 is the most frequent value)."""
    rng = np.random.default_rng(m * 7 + n + L)
    cb = (np.arange(K) - zero).astype(np.float32) / np.float32(K)
    p = np.full(K, (1 - p0) / (K - 1))
    p[K // 2] = p0
    W = rng.choice(cb, size=(m, n), p=p).astype(np.float32)
    W[m // 2] = cb[K // 2]                                         # a row without indices
    X = rng.standard_normal((n, L)).astype(np.float32)
    h = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    buf = torch.zeros(n * L + 4, device="cuda")
    Xd = buf[shift:shift + n * L]
    Xd.copy_(torch.from_numpy(X).reshape(-1))
    Y = torch.full((m, L), float("nan"), device="cuda")
    (B.cer_matmul if fmt == "cer" else B.cser_matmul)(h, Xd, Y, L)
    torch.cuda.synchronize()
    B.cer_free(h)
    want = W.astype(np.float64) @ X.astype(np.float64)
    bound = 1e-5 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64)) + 1e-30
    assert (np.abs(Y.cpu().numpy() - want) <= bound).all()


@pytest.mark.parametrize("L", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("shape", [(5, 200, 3), (300, 3000, 16), (1000, 4500, 40), (700, 9000, 5), (40, 17000, 130), (9, 36000, 4), (2100, 700, 256)])
def test_narrow_batches(shape, L):
    m, n, K = shape
    _check(m, n, L, K, 0.4, K // 2, "cer" if L % 2 else "cser")


@pytest.mark.parametrize("L", [2, 4, 7, 8])
def test_unaligned_input_and_non_zero_most_frequent_value(L):
    _check(130, 2500, L, 9, 0.6, 0, "cer", shift=1)
    _check(4100, 1030, L, 33, 0.8, 0, "cser", shift=0)


@pytest.mark.parametrize("L", [9, 11, 13, 16])
@pytest.mark.parametrize("shape", [(700, 600, 30), (520, 2900, 180), (1100, 4400, 85), (900, 9000, 60)])
def test_groups_of_columns_that_overlap(shape, L):
    m, n, K = shape
    _check(m, n, L, K, 0.35, K // 2, "cser" if L % 2 else "cer", shift=L % 3)
