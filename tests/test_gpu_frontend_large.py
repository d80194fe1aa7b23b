"""The front-end where its kernels change their form: weights and results of more than a round of the range kernel and of 128 MiB, and rows
of the sorting emitter that stay in registers or do not, one after another."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1024, 8192), (1024, 8193), (2049, 4097), (4097, 8193)])
@pytest.mark.parametrize("ends", ["first", "last"])
def test_range_and_decode(shape, ends):
    """The smallest and the largest weight at either end of the matrix, at the sizes where the range is read in another way (8 388 608
    weights) and where the result goes past the caches (33 554 432); nothing behind the result is written."""
    m, n = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    W = torch.randn((m, n), generator=g, device="cuda").clamp_(-3, 3)
    flat = W.view(-1)
    flat[0 if ends == "first" else m * n - 1], flat[1 if ends == "first" else m * n - 2] = -7.0, 8.0
    h, cb = B.cer_quantize_encode_device(W, m, n, 4, "cer")
    cb = np.asarray(cb)
    assert cb[0] == -7 and cb[-1] == 8 and len(cb) == 16   # a grid of whole numbers
    out = torch.full((m * n + 4,), float("nan"), device="cuda")
    B.cer_decode_device(h, out[:m * n].view(m, n))
    B.cer_free(h)
    assert torch.equal(out[:m * n].view(m, n), torch.round(W + 7) - 7) and torch.isnan(out[m * n:]).all()


# rows that begin anywhere in a line, shorter than a line, of one wave each and of several segments (65536 columns), with the result as far from a
# line's start; whole lines among them
@pytest.mark.parametrize("m,n,shift", [(4100, 8191, 0), (4100, 8191, 3), (4097, 8224, 0), (4097, 8224, 31), (33200, 1011, 1), (1678000, 20, 5), (600, 65003, 2)])
def test_results_past_the_caches(m, n, shift):
    """Results of 134 MB and more: the stores of a row begin at a whole line, what lies in front of it is written singly."""
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    cb = (np.arange(13) - 4).astype(np.float32)
    W = torch.tensor(cb, device="cuda")[torch.randint(0, 13, (m, n), generator=g, device="cuda", dtype=torch.int32)]
    W[torch.rand((m, n), generator=g, device="cuda") < 0.6] = 0.0
    h = B.cer_encode_device(W, m, n, cb, "cser" if n & 1 else "cer")
    out = torch.full((m * n + 64,), float("nan"), device="cuda")
    B.cer_decode_device(h, out[shift:shift + m * n].view(m, n))
    B.cer_free(h)
    assert m * n >= 1 << 25 and torch.equal(out[shift:shift + m * n].view(m, n), W)
    assert torch.isnan(out[:shift]).all() and torch.isnan(out[shift + m * n:]).all()
    B.cer_trim()


# rows of at most 12288 columns stay in registers; about 1300 workgroups take rows of 9217 and 12289 columns in turn
@pytest.mark.parametrize("shape", [(3000, 1024), (2999, 1039), (1500, 4100), (2600, 9217), (700, 12288), (1400, 12289), (300, 20001)])
@pytest.mark.parametrize("fmt", ["cer", "cser"])
def test_sorted_rows(shape, fmt):
    """The same arrays as the host encoder's; rows without an element, full rows, and rows of one value."""
    m, n = shape
    rng = np.random.default_rng(m + n)
    K = 100 if n == 9217 else 24
    cb = (np.arange(K) - 3).astype(np.float32)
    W = rng.choice(cb, size=(m, n)).astype(np.float32)
    W[rng.random((m, n)) < 0.2] = cb[40 % K]
    W[5], W[m - 1], W[m // 2] = cb[40 % K], cb[K - 1], rng.choice(cb[41 % K:], n)
    h = B.cer_encode_device(torch.from_numpy(W).cuda(), m, n, cb, fmt)
    assert B.cer_encode_sorts_rows(h, K)
    host = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    for which in (B.CER_ARRAY_OMEGA, B.CER_ARRAY_COLI, B.CER_ARRAY_OMEGAPTR, B.CER_ARRAY_ROWPTR) + ((B.CER_ARRAY_OMEGAI,) if fmt == "cser" else ()):
        assert np.array_equal(B.cer_get_array(h, which), B.cer_get_array(host, which)), which
    B.cer_free(h)
    B.cer_free(host)


@pytest.mark.parametrize("m", [2048, 2049, 2051, 2111, 2112, 2113, 8191])
@pytest.mark.parametrize("fmt", ["cer", "cser"])
def test_rows_per_wave_of_the_layout(m, fmt):
    """Row counts around the 2048 from which on a wave lays out four rows, and around the 64 of a workgroup; rows of one value among them."""
    n, K = 37, 200
    rng = np.random.default_rng(m)
    cb = (np.arange(K) - 3).astype(np.float32)
    W = cb[np.minimum(rng.geometric(0.2, size=(m, n)) - 1, K - 1)]
    W[rng.integers(0, m, 20)] = cb[0]
    W[m - 1], W[0] = cb[K - 1], cb[1]
    host = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    h = B.cer_encode_device(torch.from_numpy(W).cuda(), m, n, cb, fmt)
    for which in (B.CER_ARRAY_OMEGA, B.CER_ARRAY_COLI, B.CER_ARRAY_OMEGAPTR, B.CER_ARRAY_ROWPTR) + ((B.CER_ARRAY_OMEGAI,) if fmt == "cser" else ()):
        assert np.array_equal(B.cer_get_array(h, which), B.cer_get_array(host, which)), which
    B.cer_free(h)
    B.cer_free(host)


# (rows, columns, values, share indexed, whether a row is sorted in LDS)
SPARSE = [(300, 9217, 16, 0.05, True), (1300, 12289, 5, 0.3, True), (257, 4099, 24, 0.45, True), (20, 64512, 3, 0.02, True), (20, 64513, 3, 0.02, False),
          (300, 5000, 1, 0.0, True), (5, 20000, 256, 0.001, True), (2048, 1024, 16, 0.4, False), (3000, 2500, 250, 0.1, False)]


@pytest.mark.parametrize("case", SPARSE, ids=[f"{c[0]}x{c[1]}_K{c[2]}_{c[3]}" for c in SPARSE])
@pytest.mark.parametrize("fmt", ["cer", "cser"])
def test_mostly_implicit_rows(case, fmt):
    """Fewer than half of the elements indexed, by either kernel: the host encoder's arrays.  Rows without an element, one much longer than the
    others, nothing indexed at all."""
    m, n, K, share, sorts = case
    rng = np.random.default_rng(m + n)
    cb = (np.arange(K) - K // 2).astype(np.float32)
    W = np.where(rng.random((m, n)) < share, rng.choice(cb, size=(m, n)), np.float32(0)).astype(np.float32)
    W[m // 2] = 0.0
    W[m - 1, :n // 4], W[0, n - 1] = cb[K - 1], cb[0]
    h = B.cer_encode_device(torch.from_numpy(W).cuda(), m, n, cb, fmt)
    assert B.cer_encode_sorts_rows(h, K) == sorts
    host = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    for which in (B.CER_ARRAY_OMEGA, B.CER_ARRAY_COLI, B.CER_ARRAY_OMEGAPTR, B.CER_ARRAY_ROWPTR) + ((B.CER_ARRAY_OMEGAI,) if fmt == "cser" else ()):
        assert np.array_equal(B.cer_get_array(h, which), B.cer_get_array(host, which)), which
    B.cer_free(h)
    B.cer_free(host)
