"""Batches of 2 to 16 columns by the library's own choice (csrc/cer_narrow.hip): every number of columns per pass, 8- and 16-bit
indices, one to four tiles of groups, rows shared by several waves, rows of several windows, unaligned X, non-zero Omega[0]."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def matrix(m, n, L, K, p0, zero):
    """(W, codebook, generator); zero: position of 0 in the codebook (K // 2: 0 is the most frequent value)."""
    rng = np.random.default_rng(m * 7 + n + L)
    cb = (np.arange(K) - zero).astype(np.float32) / np.float32(K)
    p = np.full(K, (1 - p0) / (K - 1))
    p[K // 2] = p0
    W = rng.choice(cb, size=(m, n), p=p).astype(np.float32)
    W[m // 2] = cb[K // 2]                                         # a row without indices
    return W, cb, rng


def _check(m, n, L, K, p0, zero, fmt, shift=0):
    W, cb, rng = matrix(m, n, L, K, p0, zero)
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


# (m, n, K, share of the most frequent value, columns of X, columns per pass): one to four tiles of groups, 8- and 16-bit indices,
# a single wave and several per row; 0 per pass: the kernel that cer_matmul_path reports serves the batch
CHOICES = [
    (9, 36000, 4, 0.4, 8, 1), (40, 17000, 130, 0.4, 4, 1),
    (300, 3000, 16, 0.4, 2, 2), (40, 17000, 130, 0.4, 7, 2), (256, 12000, 140, 0.8, 15, 2), (300, 100, 2, 0.4, 2, 2),
    (300, 3000, 16, 0.4, 5, 4), (700, 600, 30, 0.4, 16, 4), (3000, 250, 100, 0.4, 11, 4), (1500, 1500, 200, 0.4, 3, 4),
    (2100, 700, 256, 0.4, 12, 4),
    (2100, 700, 256, 0.8, 5, 8), (2100, 700, 256, 0.8, 8, 8), (3000, 250, 100, 0.8, 13, 8), (3000, 250, 100, 0.8, 16, 8),
    (2100, 700, 256, 0.4, 13, 0), (300, 3000, 16, 0.4, 17, 0),
]


@pytest.mark.parametrize("case", CHOICES, ids=[f"{c[0]}x{c[1]}_K{c[2]}_{c[3]}_L{c[4]}_{c[5]}" for c in CHOICES])
def test_the_library_takes_the_kernel_this_file_is_about(case):
    """... with the stated number of columns per pass; that it ran shows in the rounding, which is not that of the kernel that
    cer_matmul_path reports (and is where the library does not take it)."""
    m, n, K, p0, L, columns = case
    rng = np.random.default_rng(1)
    cb = (np.arange(K) - K // 2).astype(np.float32) / np.float32(K)
    p = np.full(K, (1 - p0) / (K - 1))
    p[K // 2] = p0
    W = rng.choice(cb, size=(m, n), p=p).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    h = B.cer_encode(W, cb)
    Xd = torch.from_numpy(X).cuda()
    Y, other = (torch.full((m, L), float("nan"), device="cuda") for _ in range(2))
    assert B.cer_matmul_narrow_columns(h, L) == columns
    B.cer_matmul(h, Xd, Y, L)
    B.cer_matmul_ex(h, Xd, other, L, None, B.MatmulOpts(path=B.cer_matmul_path(h, L)))
    torch.cuda.synchronize()
    B.cer_free(h)
    assert torch.equal(Y, other) == (columns == 0)
    want = W.astype(np.float64) @ X.astype(np.float64)
    bound = 1e-5 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64)) + 1e-30
    for y in (Y, other):
        assert (np.abs(y.cpu().numpy() - want) <= bound).all()


# (m, n, K, share of the most frequent value, columns of X) around the sizes at which X and the lists of 16 waves do not fit LDS: with eight columns
# per pass those of 4, with four those of 2, ... are taken then, or 8 or 4 waves; the rounds of loads full, one more, one less.  Behind each: columns per
# pass, waves and whether they read ahead (kFew), with Omega[0] == 0 and != 0, None: another kernel (tests/test_launch_shapes.py holds the launches
# against it).
FEW = [
    ((1100, 4800, 9, 0.95, 8), None, (4, 16, False)), ((2100, 4609, 60, 0.97, 8), (4, 16, False), (4, 16, False)), ((2100, 4608, 130, 0.97, 7), None, (4, 16, False)),
    ((1100, 9728, 20, 0.95, 4), (4, 8, False), (2, 16, False)), ((1100, 9727, 9, 0.95, 3), (4, 8, False), (1, 16, False)), ((2100, 8193, 130, 0.97, 4), None, (2, 16, False)),
    ((1100, 19300, 9, 0.95, 2), (2, 8, True), (1, 16, False)), ((2100, 16385, 130, 0.97, 2), (2, 8, True), (2, 8, True)), ((2303, 19624, 3, 0.95, 4), (2, 8, True), (2, 8, True)),
    ((300, 33000, 130, 0.8, 2), (1, 8, True), (1, 8, True)), ((1100, 33000, 130, 0.95, 2), (1, 8, True), (1, 8, True)), ((300, 37000, 130, 0.8, 3), (1, 4, True), (1, 4, True)),
    ((1065, 9467, 33, 0.5, 8), (4, 8, True), (2, 16, False)), ((1303, 9428, 130, 0.5, 8), (4, 4, True), (4, 4, True)), ((1048, 9633, 130, 0.8, 12), (4, 4, True), (4, 4, True)),
    ((975, 9483, 3, 0.5, 4), (4, 8, False), (2, 16, False)), ((900, 9957, 33, 0.8, 8), (4, 4, True), (2, 16, False)), ((803, 19918, 3, 0.7, 4), (2, 4, True), (2, 4, True)),
    ((410, 38038, 3, 0.7, 3), (1, 8, True), (1, 8, True)), ((192, 18844, 64, 0.8, 2), (2, 8, True), (1, 16, False))]


@pytest.mark.parametrize("case", [f[0] for f in FEW], ids=[f"{c[0]}x{c[1]}_K{c[2]}_L{c[4]}" for c, *_ in FEW])
def test_fewer_than_16_waves(case):
    m, n, K, p0, L = case
    _check(m, n, L, K, p0, K // 2, "cser" if n % 2 else "cer", shift=n % 4)
    _check(m, n, L, K, p0, 0, "cer", shift=0)
