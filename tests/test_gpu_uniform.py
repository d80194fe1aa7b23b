"""Decode + matrix-core product of codebooks on a uniform grid (kUniform in csrc/cer_split3.hpp): with zero on the grid -- two numbers per
value -- and off it, with values that do not occur, up to 256 steps, next to values that are too far from the grid, and with values
beside it by what two binary32 roundings leave, at the edges of the tiles, against fp64."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

_steps = np.arange(-128, 128)
CODEBOOKS = {
    "zero": ((np.arange(65) - 20) / np.float32(65)).astype(np.float32),
    "offset": np.linspace(-0.31, 0.42, 64, dtype=np.float32),
    "one_side": np.linspace(0.3, 1.1, 32, dtype=np.float32),
    "gaps": (_steps[[0, 3, 100, 128, 129, 200, 255]] * np.float32(0.0173)).astype(np.float32),
    "256": (_steps * np.float32(3.1e-5) + np.float32(1e-5)).astype(np.float32),
    "ternary": np.array([-0.37, 0.0, 0.37], np.float32),
    "off_grid": np.append((_steps[::8] / np.float32(77)).astype(np.float32), np.float32(1.0003)),
}


def _beside(last, units):
    """last values of a grid of 1/77, every other one moved by so many units of its last place."""
    v = (np.arange(last + 1) / np.float32(77)).astype(np.float32)
    u = v.view(np.int32)
    u[1::2] += units * np.where(np.arange(last + 1)[1::2] % 4 == 1, 1, -1).astype(np.int32)
    return np.append(v, -v[1:]).astype(np.float32)


# values up to 2^-22 of themselves beside the grid: one unit is 2^-23 to 2^-24 of a value, eight are 2^-20 to 2^-21
CODEBOOKS["beside"] = _beside(100, 1)
CODEBOOKS["too_far"] = _beside(100, 8)
PLANES = {"zero": 2, "offset": 3, "one_side": 3, "gaps": 2, "256": 3, "ternary": 2, "off_grid": 3, "beside": 2, "too_far": 3}


@pytest.mark.parametrize("name", list(CODEBOOKS))
def test_form_and_values(name):
    """Which codebooks are two numbers, and what the pieces of a value add up to: one-hot inputs of 1 and 2 return the matrix bit for bit,
    those of 24 bits its products to 2^-23 (one rounding, and left-out products below 2^-25), by both kernels that use the pieces."""
    cb = CODEBOOKS[name]
    m, n, L = 1600, 300, 100
    rng = np.random.default_rng(5)
    W = rng.choice(cb, size=(m, n)).astype(np.float32)
    h = B.cer_encode(W, cb)
    assert B.cer_matmul_planes(h) == PLANES[name] and B.cer_matmul_fused_rows(h, L) > 0
    for first in range(0, n, L):
        at = np.arange(first, first + L)
        for full in (False, True):
            x = rng.uniform(1, 2, L).astype(np.float32) if full else rng.choice([1.0, 2.0], L).astype(np.float32)
            X = np.zeros((n, L), np.float32)
            X[at, np.arange(L)] = x
            Xd, want = torch.from_numpy(X).cuda(), W[:, at].astype(np.float64) * x
            for opts in (None, B.MatmulOpts(path=B.CER_PATH_DENSE)):
                Y = torch.full((m, L), float("nan"), device="cuda")
                B.cer_matmul(h, Xd, Y, L) if opts is None else B.cer_matmul_ex(h, Xd, Y, L, None, opts)
                torch.cuda.synchronize()
                got = Y.cpu().numpy().astype(np.float64)
                assert (np.abs(got - want) <= 2.0 ** -23 * np.abs(want)).all() if full else np.array_equal(got, want)
    B.cer_free(h)


@pytest.mark.parametrize("inputs", ["normal", "relu", "positive", "constant"])
@pytest.mark.parametrize("name", ["offset", "one_side", "256", "zero", "beside"])
@pytest.mark.parametrize("L", [60, 512])
def test_no_less_precise_than_three_pieces(name, inputs, L):
    """Inputs with a mean, where an offset's share and the integers' sum would cancel.  A value off every grid in a row that is left out
    makes the codebook three pieces."""
    m, n = 800, 3000
    rng = np.random.default_rng(L)
    cb = CODEBOOKS[name]
    near = np.argsort(np.abs(cb))[:max(3, len(cb) // 4)]  # weights near zero, as layers have them
    W = rng.choice(cb[near], size=(m, n)).astype(np.float32)
    W[1] = rng.choice(cb, size=n)
    X = rng.standard_normal((n, L)).astype(np.float32)
    X = {"normal": X, "relu": np.maximum(X, 0), "positive": np.abs(X) + np.float32(1), "constant": np.full_like(X, 0.7243)}[inputs]
    want = (W.astype(np.float64) @ X.astype(np.float64))[1:]
    scale = (np.abs(W).astype(np.float64) @ np.abs(X).astype(np.float64))[1:]
    errors = [np.linalg.norm((_product(W, cb, X)[1:] - want) / scale)]
    W[0, 0] = np.float32(0.123456789)
    errors.append(np.linalg.norm((_product(W, np.append(cb, W[0, 0]), X)[1:] - want) / scale))
    assert errors[0] <= 1.1 * errors[1], errors  # (two numbers: 0.65 of three pieces' in the mean, 1.03 at most)


def _product(W, cb, X, fmt="cer"):
    h = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
    Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
    Y = torch.full((W.shape[0], X.shape[1]), float("nan"), device="cuda")
    B.cer_matmul_ex(h, Xd, Y, X.shape[1], None, B.MatmulOpts(path=B.CER_PATH_DENSE))
    torch.cuda.synchronize()
    B.cer_free(h)
    return Y.cpu().numpy().astype(np.float64)


def _close(Y, W, X, rel=1e-6, least=0.0):
    """binary32 products and sums (as tests/test_gpu_mfma.py); least: per term, where these are subnormal."""
    W, X = W.astype(np.float64), X.astype(np.float64)
    return (np.abs(Y - W @ X) <= rel * (np.abs(W) @ np.abs(X)) + least * W.shape[1]).all()


@pytest.mark.parametrize("name", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(1, 1, 2), (255, 127, 31), (256, 128, 32), (257, 129, 33), (31, 8200, 64), (513, 640, 65),
                                   (40, 300, 130), (1100, 500, 2100)])
def test_edges_of_the_tiles(shape, name):
    m, n, L = shape
    rng = np.random.default_rng(m + n)
    W = rng.choice(CODEBOOKS[name], size=(m, n)).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    assert _close(_product(W, CODEBOOKS[name], X, "cser" if m % 2 else "cer"), W, X)


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("name", list(CODEBOOKS))
@pytest.mark.parametrize("shape", [(700, 1200, 60), (512, 4608, 512)])
def test_no_less_precise_than_fp32_products(shape, name, relu):
    """As in tests/test_gpu_mfma.py: a subnormal value, in a row that is left out, sends the matrix to the fp32 matrix cores."""
    m, n, L = shape
    rng = np.random.default_rng(n)
    cb = CODEBOOKS[name]
    W = rng.choice(cb, size=(m, n)).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    if relu:
        X = np.maximum(X, 0)
    want = (W.astype(np.float64) @ X.astype(np.float64))[1:]
    errors = [np.linalg.norm(_product(W, cb, X)[1:] - want)]
    W[0, 0] = np.float32(1e-40)
    errors.append(np.linalg.norm(_product(W, np.append(cb, W[0, 0]), X)[1:] - want))
    assert errors[0] <= errors[1], errors


@pytest.mark.parametrize("name", ["zero", "offset", "256"])
@pytest.mark.parametrize("shape", [(70, 300, 45), (2048, 1024, 2048), (2048, 260, 20)])
def test_inputs_at_the_ends_of_the_range(shape, name):
    """Infinities and NaNs as in IEEE arithmetic; inputs near the largest number, whose sum alone would overflow; and inputs whose last
    bits no bf16 number reaches (plus half of the smallest number per rounding of a subnormal sum)."""
    m, n, L = shape
    rng = np.random.default_rng(n)
    cb = CODEBOOKS[name]
    W = rng.choice(cb, size=(m, n)).astype(np.float32)
    X = rng.standard_normal((n, L)).astype(np.float32)
    X[n // 3, 1], X[n - 1, 2], X[5, 3] = np.inf, -np.inf, np.nan
    X[6, 4], X[7, 4] = np.inf, -np.inf
    Y = _product(W, cb, X)
    with np.errstate(invalid="ignore"):
        for c in (1, 2, 3, 4):
            assert np.array_equal(Y[:, c], (W.astype(np.float64) * X[:, c].astype(np.float64)).sum(1), equal_nan=True), c
    keep = np.setdiff1d(np.arange(L), [1, 2, 3, 4])
    assert _close(Y[:, keep], W, X[:, keep])
    X = rng.uniform(0.5, 1.0, (n, L)).astype(np.float32)
    W2 = W * np.float32(2.0 ** -12)
    big = X * np.float32(2.0 ** 127)
    assert _close(_product(W2, cb * np.float32(2.0 ** -12), big), W2, big)
    for k in (108, 120, 140):
        tiny = np.ldexp(X, -k).astype(np.float32)
        assert _close(_product(W, cb, tiny), W, tiny, least=5 * 2.0 ** -150), k
