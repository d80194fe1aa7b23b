"""Products from the tile index by the library's own choice (csrc/cer_tile.hip): every width of a tile, one and several bf16 pieces, buckets
of few and of many entries, groups and buckets that end early, one and several parts of W's columns, ragged sizes, unaligned X and Y,
empty and full rows, a non-zero most frequent value, infinities, NaNs and numbers down to the smallest subnormal."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B
from test_gpu_fused import _as_served, _bound, _matrix, _product

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

OFF_GRID = np.sort(np.random.default_rng(2).uniform(-1, 1, 33)).astype(np.float32)  # three pieces per value


def _prepared(W, cb, fmt="cer"):
    h = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    B.cer_prepare_strips(h)
    return h


# (m, n, L, K (0: off any grid), share of the most frequent value, zero's place in the codebook, columns per workgroup, fmt, shift)
CASES = [
    (257, 20000, 7, 4, 0.5, 0, 16, "cer", 0), (1601, 700, 47, 16, 0.5, 8, 16, "cser", 1), (1999, 999, 130, 64, 0.5, 32, 32, "cer", 3),
    (500, 3000, 191, 16, 0.7, 8, 48, "cser", 2), (900, 6001, 33, 32, 0.8, 0, 48, "cer", 1), (1030, 12001, 63, 16, 0.5, 8, 64, "cser", 0),
    (513, 9000, 250, 64, 0.4, 0, 64, "cer", 2), (130, 4000, 99, 4, 0.4, 0, 16, "cser", 0), (257, 20000, 13, 3, 0.5, 1, 16, "cer", 1),
    (1601, 700, 191, 17, 0.5, 8, 32, "cser", 0), (900, 6001, 95, 33, 0.8, 16, 48, "cer", 3), (1030, 12001, 130, 7, 0.5, 0, 48, "cser", 0),
    (1999, 999, 250, 63, 0.5, 0, 32, "cer", 1), (900, 6001, 31, 0, 0.4, 0, 32, "cser", 0), (513, 9000, 65, 0, 0.4, 0, 64, "cer", 1),
    (1601, 700, 401, 0, 0.4, 0, 64, "cser", 2), (4096, 9216, 99, 32, 0.85, 16, 64, "cser", 0),
]


def _case(m, n, K, p0, zero):
    if K:
        return _matrix(m, n, K, p0, zero, m + n)
    rng = np.random.default_rng(m + n)
    W = rng.choice(OFF_GRID, size=(m, n), p=[p0] + [(1 - p0) / 32] * 32).astype(np.float32)
    W[m // 2] = OFF_GRID[0]
    return W, OFF_GRID, rng


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}_L{c[2]}_K{c[3]}" for c in CASES])
def test_products(case):
    """Also: not further from fp64 than the gathers (2-norm), whose sums are products in binary32, nor than the decoded matrix."""
    m, n, L, K, p0, zero, columns, fmt, shift = case
    W, cb, rng = _case(m, n, K, p0, zero)
    X = rng.standard_normal((n, L)).astype(np.float32)
    h = _prepared(W, cb, fmt)
    assert B.cer_matmul_tile_columns(h, L) == columns and B.cer_matmul_fused_rows(h, L) == 0 and B.cer_matmul_planes(h) == (3 if K == 0 else 1 if K in (4, 16, 32, 64) else 2)
    want = W.astype(np.float64) @ X.astype(np.float64)
    Y = _product(h, X, m, L, shift, fmt=fmt)
    assert (np.abs(Y - want) <= 0.1 * _bound(W, X)).all()
    err = [np.linalg.norm(y - want) for y in (Y, *(_product(h, X, m, L, opts=B.MatmulOpts(path=p)) for p in (B.CER_PATH_GEMM, B.CER_PATH_DENSE)))]
    assert err[0] <= err[1] and err[0] <= err[2], err
    B.cer_free(h)


def test_rows_of_very_different_length():
    rng = np.random.default_rng(3)
    m, n, L = 1200, 5000, 130
    cb = np.array([0.0, 0.5, -0.25, 1.0], np.float32)
    W = np.where(rng.random((m, n)) < rng.choice([0.0, 0.1, 0.5, 1.0], size=(m, 1)), rng.choice(cb[1:], size=(m, n)), np.float32(0)).astype(np.float32)
    W[:, 640:1280] = 0
    W[64:128] = 0
    X = rng.standard_normal((n, L)).astype(np.float32)
    h = _prepared(W, cb)
    assert B.cer_matmul_tile_columns(h, L) > 0
    Y = _product(h, X, m, L)
    B.cer_free(h)
    assert (np.abs(Y - W.astype(np.float64) @ X.astype(np.float64)) <= _bound(W, X)).all()
    assert (Y[~W.any(1)] == 0).all()


# calls that the gathers, the strips and the decoded matrix serve without the index; one to three pieces
REPEATED = [(1601, 700, 47, 16, 0.5, 8), (300, 1000, 31, 16, 0.5, 0), (500, 3000, 191, 13, 0.7, 6), (900, 6001, 33, 32, 0.8, 16), (257, 20000, 17, 3, 0.5, 0),
            (1030, 12001, 63, 16, 0.5, 8), (1999, 999, 250, 63, 0.5, 0), (900, 6001, 31, 0, 0.4, 0), (513, 9000, 130, 0, 0.4, 0)]


@pytest.mark.parametrize("case", REPEATED, ids=[f"{c[0]}x{c[1]}_L{c[2]}_K{c[3]}" for c in REPEATED])
def test_rows_formed_again(case):
    """Infinities and NaNs count as in the kernel that is replaced, in every row of the matrix and no other column; what stays finite is as
    close as ever; so are inputs below 2^-110 in some or all of X."""
    m, n, L, K, p0, zero = case
    W, cb, rng = _case(m, n, K, p0, zero)
    W[m // 3, : n // 2] = cb[K // 2]
    h = _prepared(W, cb)
    omega0, path = float(B.cer_get_array(h, B.CER_ARRAY_OMEGA)[0]), B.cer_matmul_path(h, L)
    assert B.cer_matmul_tile_columns(h, L) > 0
    X = rng.standard_normal((n, L)).astype(np.float32)
    X[n // 3, 1], X[n - 1, L - 1], X[5, 3], X[6, 4], X[7, 4], X[0, 6], X[n // 2, 6] = np.inf, -np.inf, np.nan, np.inf, -np.inf, -np.inf, -np.inf
    odd = [1, 3, 4, 6, L - 1]
    Y, want = _product(h, X, m, L), _as_served(W, X[:, odd], omega0, path)
    assert np.array_equal(np.isfinite(Y[:, odd]), np.isfinite(want))
    bad = ~np.isfinite(want)
    assert np.array_equal(Y[:, odd][bad], want[bad].astype(np.float32), equal_nan=True)
    finite = np.where(np.isfinite(X), X, 0)  # (rows that do not index an infinity: the rest of the column)
    bound = _bound(W, finite) * (1 + (abs(omega0) > 0) * 4) + 1e-5 * abs(omega0) * np.abs(finite).sum(0)
    close = np.abs(Y - W.astype(np.float64) @ finite.astype(np.float64)) <= bound
    keep = np.setdiff1d(np.arange(L), odd)
    assert close[:, keep].all() and close[:, odd][~bad].all()
    for tiny in (np.ones((1, L), bool), np.arange(L)[None, :] % 2 == 0, rng.random((n, L)) < 0.5):
        Z = np.where(tiny, np.ldexp(finite, -121), finite).astype(np.float32)
        bound = 1e-5 * (np.abs(W).astype(np.float64) @ np.abs(Z).astype(np.float64) + abs(omega0) * np.abs(Z.astype(np.float64)).sum(0)) + n * 2.0 ** -150
        assert (np.abs(_product(h, Z, m, L) - W.astype(np.float64) @ Z.astype(np.float64)) <= bound).all()
    B.cer_free(h)


def test_replayed_from_a_graph():
    m, n, L, K = 1030, 12001, 63, 16
    W, cb, rng = _matrix(m, n, K, 0.5, K // 2, 1)
    h = _prepared(W, cb)
    assert B.cer_matmul_tile_columns(h, L) > 0
    X, Y = torch.zeros((n, L), device="cuda"), torch.zeros((m, L), device="cuda")
    B.cer_matmul(h, X, Y, L)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.cer_matmul(h, X, Y, L, torch.cuda.current_stream())
    for rep in range(3):
        X.copy_(torch.from_numpy(rng.standard_normal((n, L)).astype(np.float32)))
        g.replay()
        torch.cuda.synchronize()
        eager = torch.empty_like(Y)
        B.cer_matmul(h, X, eager, L)
        torch.cuda.synchronize()
        assert torch.equal(Y, eager), rep
    B.cer_free(h)


# codebooks whose numbers come with both signs: one piece, two numbers, three pieces
SYMMETRIC = {"one_piece": (np.arange(16) - 8).astype(np.float32), "grid": (np.arange(35) - 17).astype(np.float32) / np.float32(17) * 8,
             "three_pieces": np.sort(np.concatenate([[0.0], s := np.random.default_rng(4).uniform(0.1, 8, 16), -s])).astype(np.float32)}


@pytest.mark.parametrize("name,m,n,L", [("one_piece", 1601, 700, 47), ("one_piece", 900, 9000, 130), ("grid", 1601, 700, 191), ("grid", 1030, 12001, 130),
                                        ("three_pieces", 1601, 700, 401), ("three_pieces", 513, 9000, 130)])
def test_large_inputs_that_cancel(name, m, n, L):
    """Sums that are zero or small because large terms cancel, next to inputs whose last bits no piece has (in the same column and in others):
    they are what the terms give, exact where those are, whatever is formed again; so are sums of inputs near the largest number."""
    cb = SYMMETRIC[name]
    rng = np.random.default_rng(m)
    W = np.where(rng.random((m, n)) < 0.5, rng.choice(cb, size=(m, n)), np.float32(0)).astype(np.float32)
    a, b, c, d = n // 3, n // 3 + 1, n - 1, 0
    W[::7] = 0
    v = rng.choice(cb[cb > 0], size=W[::7].shape[0])
    W[::7, a], W[::7, b] = v, -v
    W[::14, c], W[::14, d] = cb[0], cb[-1]       # such a row's faint terms
    h = _prepared(W, cb)
    assert B.cer_matmul_tile_columns(h, L) > 0 and B.cer_matmul_planes(h) == {"one_piece": 1, "grid": 2, "three_pieces": 3}[name]
    W64 = W.astype(np.float64)
    X = rng.standard_normal((n, L)).astype(np.float32)
    for j, e in enumerate((40, 61, 62, 63, 64, 80, 100, 120)):
        X[a, j] = np.ldexp(1.0, e)
    X[b], X[c], X[d] = X[a], 0, 0
    for lossy in (False, True):
        if lossy:
            X[c], X[d] = np.ldexp(1.2345, -130), np.ldexp(-1.7, -140)
        Y, want = _product(h, X, m, L), W64 @ X.astype(np.float64)
        assert np.isfinite(Y).all()
        # those rows are the two faint terms, which a binary32 sum may also have lost next to the large ones
        tiny, size = W64[::7][:, [c, d]] @ X[[c, d]].astype(np.float64), np.abs(W64[::7][:, [c, d]]) @ np.abs(X[[c, d]]).astype(np.float64)
        assert (np.abs(Y[::7] - tiny) <= np.where(np.arange(L) < 8, 1, 1e-5) * size + 2.0 ** -148).all()
        keep = np.arange(m) % 7 != 0
        assert (np.abs(Y - want) <= _bound(W, X))[keep].all()
    for scale in (2.0 ** 112, 2.0 ** -118):
        Z = (np.abs(X) * (np.abs(X) < 8) * scale).astype(np.float32)
        assert (np.abs(_product(h, Z, m, L) - W64 @ Z.astype(np.float64)) <= 1e-5 * (np.abs(W64) @ Z.astype(np.float64)) + n * 2.0 ** -150).all()
    Z = np.zeros((n, L), np.float32)             # numbers that round to an infinite bf16 one, times the smallest value
    Z[np.arange(L) * 5 % n, np.arange(L)] = 3.4e38
    with np.errstate(over="ignore"):
        want = (W64 @ Z.astype(np.float64)).astype(np.float32)
    Y = _product(h, Z, m, L)
    assert np.array_equal(np.isfinite(Y), np.isfinite(want)) and np.allclose(Y, want, rtol=1e-6, atol=0)
    B.cer_free(h)


# (codebook, m, n, share of indexed elements, L, columns per workgroup, rows per workgroup of decode + product in one launch without the index)
WIDE = [("one_piece", 200, 64990, 0.5, 41, 16, 0), ("one_piece", 300, 40000, 0.15, 99, 48, 0), ("one_piece", 700, 4000, 0.5, 99, 64, 16),
        ("grid", 200, 64990, 0.5, 130, 48, 0), ("grid", 640, 25088, 0.4, 99, 48, 16), ("three_pieces", 300, 40000, 0.15, 200, 64, 16)]


@pytest.mark.parametrize("name,m,n,indexed,L,columns,fused", WIDE)
def test_long_sums(name, m, n, indexed, L, columns, fused):
    """Rows up to the widest, where a wave's running sums are longest (an eighth of a part of W's columns for one piece and for grids): not
    further from fp64 (2-norm) than the strips, the gathers, or decode + product in one launch where that is what runs without the index.  X of one
    sign: the result's rounding, 0.58 of 2^-24 at most in the root of the mean square, and as much for the waves' sums and their running sums
    before them together make no more than 2^-24 unless the latter grow with n."""
    cb = {"one_piece": (np.arange(17) - 8).astype(np.float32) / 8, "grid": ((np.arange(35) - 17) * np.float32(0.0123)).astype(np.float32)}.get(name, OFF_GRID)
    zero = int(np.argmin(np.abs(cb)))
    rng = np.random.default_rng(n + L)
    W = np.where(rng.random((m, n), dtype=np.float32) < indexed, cb[rng.integers(0, len(cb), size=(m, n))], cb[zero]).astype(np.float32)
    h, plain = _prepared(W, cb), B.cer_encode(W, cb)
    assert B.cer_matmul_tile_columns(h, L) == columns and B.cer_matmul_fused_rows(plain, L) == fused
    W64, normal = W.astype(np.float64), rng.standard_normal((n, L), dtype=np.float32)
    for X in (normal, np.abs(normal) + np.float32(1)):
        want = W64 @ X.astype(np.float64)
        err = np.linalg.norm(_product(h, X, m, L) - want)
        for other in (_product(h, X, m, L, opts=B.MatmulOpts(path=B.CER_PATH_STRIP)), _product(h, X, m, L, opts=B.MatmulOpts(path=B.CER_PATH_GEMM)),
                      *([_product(plain, X, m, L)] if fused else [])):
            assert err <= np.linalg.norm(other - want)
        assert X is normal or err <= 2.0 ** -24 * np.linalg.norm(want)
    B.cer_free(h)
    B.cer_free(plain)
