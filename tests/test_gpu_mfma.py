"""Decode + matrix-core product over bf16 pieces (csrc/cer_mfma.hip): codebooks of one, two and three pieces at the edges of
its tiles (256 rows, 32 or 64 columns, steps of 32 / 64 and rounds of 128 columns of W), against fp64 on the host."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CODEBOOKS = {  # significands of 8, 16 and 24 bits
    "one": np.array([0.0, 1.0, -0.75, 3.0], np.float32),
    "two": np.array([0.0, 1.0, -0.3330078125, 1.0009765625], np.float32),
    "three": np.array([0.0, 1.0, -1.0 / 3.0, 0.1], np.float32),
}


def _product(W, cb, X, fmt="cer"):
    h = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    Xd = torch.from_numpy(X).cuda()
    Y = torch.full((W.shape[0], X.shape[1]), float("nan"), device="cuda")
    B.cer_matmul_ex(h, Xd, Y, X.shape[1], None, B.MatmulOpts(path=B.CER_PATH_DENSE))
    torch.cuda.synchronize()
    B.cer_free(h)
    return Y.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("pieces", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(1, 1, 2), (255, 127, 31), (256, 128, 32), (257, 129, 33), (31, 8200, 64), (513, 640, 65), (40, 300, 130)])
def test_edges_of_the_tiles(shape, pieces):
    m, n, L = shape
    rng = np.random.default_rng(m + n)
    cb = CODEBOOKS[pieces]
    W = rng.choice(cb, size=(m, n), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    Y = _product(W, cb, X, "cser" if m % 2 else "cer")
    want = W.astype(np.float64) @ X.astype(np.float64)
    # the bound of binary32 products and sums, with room for a few of the latter
    assert (np.abs(Y - want) <= 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64))).all()


def test_inputs_that_have_no_three_pieces():
    """Infinities, NaNs and numbers that round to an infinite bf16: what fp32 gives."""
    cb = np.array([1.0, 0.5], np.float32)
    rng = np.random.default_rng(1)
    W = rng.choice(cb, size=(64, 256)).astype(np.float32)
    X = rng.standard_normal((256, 40)).astype(np.float32)
    X[3, 5], X[7, 6], X[200, 7], X[255, 8] = np.inf, -np.inf, np.nan, 3.4e38
    Y = _product(W, cb, X)
    assert (Y[:, 5] == np.inf).all() and (Y[:, 6] == -np.inf).all() and np.isnan(Y[:, 7]).all()
    assert np.allclose(Y[:, 8], W[:, 255] * np.float64(X[255, 8]), rtol=1e-6)
    keep = np.r_[0:5, 9:40]
    want = W.astype(np.float64) @ X[:, keep].astype(np.float64)
    assert (np.abs(Y[:, keep] - want) <= 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X[:, keep]).astype(np.float64))).all()


# (70, 300, 45): the small tiles; (2048, 1024, 2048): those of 256 rows; (2048, 260, 20): their 32-column form or the small one
@pytest.mark.parametrize("pieces", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(70, 300, 45), (2048, 1024, 2048), (2048, 260, 20)])
def test_infinities_and_nans(shape, pieces):
    """A column with infinities or a NaN is what the dense product gives in IEEE arithmetic, for codebooks of every kind: infinite
    under a non-zero weight, NaN under a zero one or where two infinities meet; the other columns are untouched."""
    m, n, L = shape
    rng = np.random.default_rng(n)
    W = rng.choice(CODEBOOKS[pieces], size=(m, n), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    X[n // 3, 1], X[n - 1, 2], X[5, 3] = np.inf, -np.inf, np.nan
    X[6, 4], X[7, 4], X[8, 9] = np.inf, -np.inf, np.inf
    Y = _product(W, CODEBOOKS[pieces], X)
    special = [1, 2, 3, 4, 9]
    with np.errstate(invalid="ignore"):
        for c in special:
            want = (W.astype(np.float64) * X[:, c].astype(np.float64)).sum(1)
            assert not np.isfinite(want).any()
            assert np.array_equal(Y[:, c], want, equal_nan=True), c
    keep = np.setdiff1d(np.arange(L), special)
    want = W.astype(np.float64) @ X[:, keep].astype(np.float64)
    assert (np.abs(Y[:, keep] - want) <= 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X[:, keep]).astype(np.float64))).all()


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("pieces", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(700, 1200, 60), (2000, 500, 300), (512, 4608, 512)])
def test_no_less_precise_than_fp32_products(shape, pieces, relu):
    """Against fp64, in the 2-norm: not further off than the fp32 matrix cores, which serve the same matrix when one of its values has
    no pieces (a subnormal one, in a row that is left out here)."""
    m, n, L = shape
    rng = np.random.default_rng(n)
    cb = CODEBOOKS[pieces]
    W = rng.choice(cb, size=(m, n), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    if relu:
        X = np.maximum(X, 0)
    want = (W.astype(np.float64) @ X.astype(np.float64))[1:]
    errors = [np.linalg.norm(_product(W, cb, X)[1:] - want)]
    W[0, 0] = np.float32(1e-40)
    errors.append(np.linalg.norm(_product(W, np.append(cb, W[0, 0]), X)[1:] - want))
    assert errors[0] <= errors[1], errors


def _tiny_cases():
    """Inputs of one size (2^-k times normal ones), inputs over 140 powers of two in one column, and inputs of ordinary size that a
    third of W's rows does not touch -- what these rows see is tiny."""
    rng = np.random.default_rng(17)
    for m, n, L in ((70, 300, 45), (2048, 1024, 2048), (2048, 260, 20)):
        for k in (100, 108, 112, 120, 128, 140, 147):
            yield f"{m}x{n}x{L} 2^-{k}", m, n, np.ldexp(rng.standard_normal((n, L)), -k).astype(np.float32), None
        X = np.ldexp(rng.standard_normal((n, L)), -rng.integers(5, 146, size=(n, 1))).astype(np.float32)
        yield f"{m}x{n}x{L} mixed", m, n, X, None
        X = np.ldexp(rng.standard_normal((n, L)), -118).astype(np.float32)
        X[::4] = rng.standard_normal(X[::4].shape)
        X[1, 7], X[n - 1, 8] = np.float32(1e38), -np.inf  # together with what the other part of the repetition is for (3e38 is finite)
        yield f"{m}x{n}x{L} rows apart", m, n, X, slice(0, None, 4)


@pytest.mark.parametrize("pieces", list(CODEBOOKS))
def test_inputs_with_bits_below_the_smallest_piece(pieces):
    """Numbers whose last bits no bf16 number reaches (below 2^-110), down to the smallest subnormal, keep all of them: the bound of
    binary32 products and sums, plus half of the smallest number for each of the n roundings of a sum that is subnormal itself
    (and as much for each of the matrix instruction's partial products, at most 6)."""
    cb = CODEBOOKS[pieces]
    rng = np.random.default_rng(23)
    for name, m, n, X, apart in _tiny_cases():
        W = rng.choice(cb, size=(m, n), p=[0.1, 0.3, 0.3, 0.3]).astype(np.float32)
        if apart is not None:
            W[::3, apart] = 0.0
        Y = _product(W, cb, X)
        with np.errstate(invalid="ignore"):
            want = W.astype(np.float64) @ X.astype(np.float64)
            bound = 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64)) + 7 * n * 2.0 ** -150
        odd = ~np.isfinite(want)
        assert np.array_equal(Y[odd], want[odd], equal_nan=True), name
        assert (np.abs(Y[~odd] - want[~odd]) <= bound[~odd]).all(), (name, np.nanmax((np.abs(Y - want) / bound)[~odd]))


@pytest.mark.parametrize("pieces", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(70, 300, 45), (2048, 1024, 2048)])
def test_empty_rows_and_columns(shape, pieces):
    """Sums that are exactly zero -- rows of W without an element, columns of X without one -- beside ordinary ones."""
    m, n, L = shape
    rng = np.random.default_rng(m)
    W = rng.choice(CODEBOOKS[pieces], size=(m, n), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    W[::9], X[:, ::7] = 0.0, 0.0
    Y = _product(W, CODEBOOKS[pieces], X)
    assert (Y[::9] == 0).all() and (Y[:, ::7] == 0).all()
    want = W.astype(np.float64) @ X.astype(np.float64)
    assert (np.abs(Y - want) <= 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64))).all()


@pytest.mark.parametrize("pieces", list(CODEBOOKS))
def test_nothing_behind_the_inputs_reaches_the_result(pieces):
    """NaNs right behind X, and the step of the kernels that crosses its end."""
    rng = np.random.default_rng(5)
    cb = CODEBOOKS[pieces]
    for m, n, L in ((300, 130, 70), (64, 257, 33), (500, 1027, 3)):
        W = rng.choice(cb, size=(m, n), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
        X = rng.standard_normal((n, L)).astype(np.float32)
        buf = torch.full((n * L + 200 * L,), float("nan"), device="cuda")
        buf[:n * L].copy_(torch.from_numpy(X).reshape(-1))
        h = B.cer_encode(W, cb)
        Y = torch.full((m, L), float("nan"), device="cuda")
        B.cer_matmul_ex(h, buf, Y, L, None, B.MatmulOpts(path=B.CER_PATH_DENSE))
        torch.cuda.synchronize()
        B.cer_free(h)
        want = W.astype(np.float64) @ X.astype(np.float64)
        assert (np.abs(Y.cpu().numpy() - want) <= 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64))).all()


@pytest.mark.parametrize("pieces", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(512, 4500, 640), (1100, 1300, 500), (64, 5000, 45), (300, 2200, 20), (512, 3100, 1000), (58000, 50, 10), (289, 33, 1000), (1030, 3100, 2000)])
def test_parts_of_unequal_length(shape, pieces):
    """Splits along n that do not divide it, with a workgroup's outputs once more in binary32 where X asks for it: one column of zeros, one of
    inputs with bits below the smallest piece, an infinity in the last row.  Bounds as above.  (1030, 3100, 2000): the last part has an odd
    number of steps, and the last tile of rows ends where the pieces of W do."""
    m, n, L = shape
    rng = np.random.default_rng(n)
    W = rng.choice(CODEBOOKS[pieces], size=(m, n), p=[0.4, 0.2, 0.2, 0.2]).astype(np.float32)
    plain = rng.standard_normal((n, L)).astype(np.float32)
    for what in ("plain", "zeros", "tiny", "infinite"):
        X = plain.copy()
        if what == "zeros":
            X[:, 3] = 0.0
        if what == "tiny":
            X[:, 3], X[:, L - 1] = 0.0, X[:, L - 1] * np.float32(2.0 ** -125)
        if what == "infinite":
            X[n - 1, L - 2] = np.inf
        Y = _product(W, CODEBOOKS[pieces], X)
        with np.errstate(invalid="ignore"):
            want = W.astype(np.float64) @ X.astype(np.float64)
            bound = 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64)) + 7 * n * 2.0 ** -150
        odd = ~np.isfinite(want)
        assert np.array_equal(Y[odd], want[odd], equal_nan=True), what
        assert (np.abs(Y[~odd] - want[~odd]) <= bound[~odd]).all(), what


@pytest.mark.parametrize("pieces,m,n,L,fused", [("one", 200, 64990, 99, False), ("two", 200, 64990, 41, False), ("three", 200, 64990, 200, False),
                                                ("grid", 200, 64990, 41, False), ("three", 300, 40000, 41, True)])
def test_sums_of_many_parts_are_rounded_once(pieces, m, n, L, fused):
    """Terms of one sign, so that the parts of W's columns add up to much more than each of them: they are added in binary64, and what is left is
    the rounding of the result, 2^-24 of it at most and 0.58 of that in the root of the mean square, and the parts' own errors, which are
    smaller by the root of their number.  (Added in binary32: 0.73 to 1.2 of 2^-24.)  2-norm."""
    rng = np.random.default_rng(n + L)
    cb = {"one": np.arange(9) / 8, "two": np.sort(rng.choice(np.arange(257, 32768), 23, replace=False) | 1) / 32768, "three": np.sort(rng.uniform(0, 1, 23)),
          "grid": np.arange(18) * np.float32(0.0123)}[pieces].astype(np.float32)
    if cb[0] != 0:
        cb = np.concatenate([np.zeros(1, np.float32), cb])
    W = np.where(rng.random((m, n), dtype=np.float32) < (0.15 if fused else 0.5), cb[rng.integers(1, len(cb), size=(m, n))], np.float32(0))
    X = np.abs(rng.standard_normal((n, L), dtype=np.float32)) + 1
    h = B.cer_encode(W, cb)
    assert B.cer_matmul_planes(h) == {"one": 1, "two": 2, "three": 3, "grid": 2}[pieces]
    Y = torch.empty((m, L), device="cuda")
    if fused:
        assert B.cer_matmul_fused_rows(h, L) > 0
        B.cer_matmul(h, torch.from_numpy(X).cuda(), Y, L)
    else:
        B.cer_matmul_ex(h, torch.from_numpy(X).cuda(), Y, L, None, B.MatmulOpts(path=B.CER_PATH_DENSE))
    torch.cuda.synchronize()
    B.cer_free(h)
    want = W.astype(np.float64) @ X.astype(np.float64)
    assert np.linalg.norm(Y.cpu().numpy() - want) <= 2 / 3 * 2.0 ** -24 * np.linalg.norm(want)


# The decoder's ranks and what the product looks up for them, both tiles, and wide batches where pieces take their place: rows of more columns than
# a segment of eight or four rows holds (6144, 12288; one segment of 33792 behind them), two rows per workgroup, remainders of 32 columns and rows,
# all 256 ranks.
def _grid(K):
    return (np.arange(K) - K // 2).astype(np.float32) / np.float32(K / 2.0)


# Behind each case: rows per workgroup of the decoder and its threads, whether it leaves ranks, whether the product's tile is the large one
# (tests/test_launch_shapes.py holds the launches against it).
RANKS = [
    (("three", 1300, 200, 100), (4, 512, True, False)), (("three", 1300, 200, 1897), (4, 512, False, True)),
    (("grid113", 2200, 700, 128), (8, 512, True, False)), (("grid113", 2200, 700, 1289), (8, 512, False, True)),
    (("two", 33, 500, 24), (4, 512, True, False)), (("two", 33, 500, 2025), (4, 512, True, False)),
    (("two", 600, 500, 2025), (4, 512, False, False)), (("two", 1200, 500, 2025), (4, 512, False, True)),
    (("any256", 290, 777, 66), (4, 512, False, True)), (("grid113", 37, 6144, 40), (4, 512, False, False)),
    (("any256", 67, 6145, 33), (4, 512, False, False)), (("three", 1100, 6177, 34), (4, 512, True, False)),
    (("two", 600, 12288, 5), (4, 512, True, False)), (("any256", 520, 12289, 20), (4, 1024, True, False)),
    (("two", 5, 33792, 20), (2, 1024, True, False)), (("grid113", 3, 33793, 70), (4, 1024, False, False)),
    (("any256", 33, 13000, 40), (4, 1024, False, True)), (("one", 19, 6200, 35), (4, 512, False, False)),
    (("one", 9, 12300, 35), (4, 1024, False, False)), (("any256", 515, 70001, 3), (4, 1024, True, False)),
    (("two", 1300, 6200, 130), (4, 512, True, True)), (("any256", 1300, 6200, 130), (4, 512, True, True)),
    (("grid113", 1301, 6200, 130), (4, 512, True, True)), (("any256", 600, 13000, 150), (4, 1024, True, True))]


def rank_case(name, m, n, L):
    """(W, codebook, whether it is a CSER matrix, generator)"""
    rng = np.random.default_rng(m * L)
    cb = {"grid113": _grid(113), "any256": np.sort(rng.standard_normal(256)).astype(np.float32)}.get(name, CODEBOOKS.get(name))
    p = np.full(len(cb), 0.5 / (len(cb) - 1))
    p[len(cb) // 2] = 0.5
    return rng.choice(cb, size=(m, n), p=p).astype(np.float32), cb, m % 2 == 1, rng


@pytest.mark.parametrize("case", [case for case, _ in RANKS])
def test_ranks_and_the_lines_of_their_choice(case):
    name, m, n, L = case
    W, cb, cser, rng = rank_case(*case)
    X = rng.standard_normal((n, L)).astype(np.float32)
    Y = _product(W, cb, X, "cser" if cser else "cer")
    want = W.astype(np.float64) @ X.astype(np.float64)
    assert (np.abs(Y - want) <= 1e-6 * (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64))).all()
    X[n // 3, 1], X[n - 1, 0] = np.inf, np.nan  # the products in binary32 take their weights from the ranks as well
    Y = _product(W, cb, X, "cser" if cser else "cer")
    with np.errstate(invalid="ignore"):
        want = W.astype(np.float64) @ X.astype(np.float64)
        scale = np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64)
    assert (np.isnan(Y) == np.isnan(want)).all() and np.isnan(Y[:, 0]).all()
    inf = np.isinf(want)
    assert (Y[inf] == want[inf]).all()
    fine = np.isfinite(want)
    assert (np.abs(Y[fine] - want[fine]) <= 1e-6 * scale[fine]).all()
