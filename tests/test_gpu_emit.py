"""The device encoder's two emitters (csrc/frontend.hip): every array of a handle encoded on the device is that of the host's encoder,
for rows that are sorted in LDS (half or more of the elements indexed, 1024 columns or more, the longest row's indices within LDS) and
for those that are not: widths around the runs of 16 columns per lane, one to 256 values, rows without indices and full ones, rows that
begin at every place of a 16-byte line, and rows of which the half that is indexed just fits and just does not."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ARRAYS = (B.CER_ARRAY_COLI, B.CER_ARRAY_OMEGAPTR, B.CER_ARRAY_ROWPTR, B.CER_ARRAY_OMEGA, B.CER_ARRAY_COUNT)


# (m, n, K, share of the most frequent value)
CASES = [(40, 1023, 5, 0.3), (40, 1024, 5, 0.3), (33, 1025, 64, 0.2), (21, 1039, 9, 0.4), (9, 2047, 256, 0.1), (9, 2048, 256, 0.1), (300, 9000, 100, 0.25),
         (2000, 1100, 7, 0.4), (30, 4097, 2, 0.5), (5, 64512, 30, 0.3), (5, 64513, 30, 0.3), (600, 3000, 200, 0.1), (12, 1500, 33, 0.9)]


SORTED = {(40, 1023): False, (40, 1024): True, (33, 1025): True, (21, 1039): True, (9, 2047): True, (9, 2048): True, (300, 9000): True, (5, 64513): False}


@pytest.mark.parametrize("fmt", ["cer", "cser"])
@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}_K{c[2]}_{c[3]}" for c in CASES])
def test_arrays_equal_the_host_encoders(case, fmt):
    m, n, K, p0 = case
    rng = np.random.default_rng(n + K)
    cb = ((np.arange(K) - K // 2) / np.float32(K)).astype(np.float32)
    p = np.full(K, (1 - p0) / (K - 1))
    p[K // 2] = p0
    W = rng.choice(cb, size=(m, n), p=p).astype(np.float32)
    W[m // 2] = cb[K // 2]          # no indices
    W[m - 1] = cb[0]                # one group, every column
    W[1, :n // 2] = cb[K - 1]
    _check(W, cb, fmt, SORTED.get((m, n)))


def _check(W, cb, fmt, sorted_rows):
    m, n = W.shape
    hh = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    if sorted_rows is not None:
        assert B.cer_encode_sorts_rows(hh, len(cb)) == sorted_rows
    hd = B.cer_encode_device(torch.from_numpy(W).cuda(), m, n, cb, fmt)
    for which in ARRAYS + ((B.CER_ARRAY_OMEGAI,) if fmt == "cser" else ()):
        assert np.array_equal(B.cer_get_array(hd, which), B.cer_get_array(hh, which)), which
    out = torch.empty((m, n), device="cuda")
    B.cer_decode_device(hd, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), W)
    B.cer_free(hh)
    B.cer_free(hd)


# the longest row's indices and the counters of 5 values: 2 * longest + 16 rounded up to 16, + 256 + 8 * 33 * 4 bytes; 65536 at most
LONGEST = 32096


@pytest.mark.parametrize("fmt", ["cer", "cser"])
@pytest.mark.parametrize("n", [60000, 64160])
@pytest.mark.parametrize("longest", [LONGEST, LONGEST + 16])
def test_widest_rows(n, longest, fmt):
    """Half of a row or more is indexed and just fits LDS, or just does not: slots beyond 32767, in both halves of the counters."""
    m, K = 5, 5
    rng = np.random.default_rng(n + longest)
    cb = np.array([0, 0.25, -0.5, 0.75, 1.0], np.float32)
    W = np.zeros((m, n), np.float32)
    for r in range(m):
        count = longest - 3 * r if n < 2 * (longest - 16) else longest
        W[r, rng.permutation(n)[:count]] = rng.choice(cb[1:], size=count, p=(0.6, 0.2, 0.15, 0.05))
    W[2, : n - longest] = 0.0      # the implicit value first, then nothing else
    W[2, n - longest:] = rng.choice(cb[1:], size=longest)
    _check(W, cb, fmt, longest == LONGEST)
