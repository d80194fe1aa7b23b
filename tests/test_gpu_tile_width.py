"""Choice of the tile width of the kernel that gathers from L2 (pick_wide_tile in csrc/cer_gemm.hip)."""
import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# columns per tile where rows of X are not whole lines: the widest tile while it holds the whole batch, however large X is; narrow ones
# for wide batches of a large X; the tile of 64 columns where it holds the batch
@pytest.mark.parametrize("case", [(1024, 25088, 100, 128), (1024, 25088, 200, 32), (1024, 4096, 60, 64)])
def test_tile_width_of_wide_batches(case):
    """The library's choice among 32, 64 and 128 columns per tile, told by the rounding: every width sums in an order of its own."""
    m, n, L, want = case
    rng = np.random.default_rng(n + L)
    cb = np.array([0.0, 1.0, -0.5, 0.25], np.float32)
    W = np.where(rng.random((m, n)) < 0.05, rng.choice(cb[1:], size=(m, n)), np.float32(0)).astype(np.float32)
    X = torch.from_numpy(rng.standard_normal((n, L)).astype(np.float32)).cuda()
    h = B.cer_encode(W, cb)
    Y = {}
    for cols in (0, 32, 64, 128):
        Y[cols] = torch.full((m, L), float("nan"), device="cuda")
        B.cer_matmul_ex(h, X, Y[cols], L, None, B.MatmulOpts(path=B.CER_PATH_GEMM, tile_cols=cols))
    torch.cuda.synchronize()
    B.cer_free(h)
    assert [cols for cols in (32, 64, 128) if torch.equal(Y[0], Y[cols])] == [want]
    ref = W.astype(np.float64) @ X.cpu().numpy().astype(np.float64)
    bound = 1e-5 * (np.abs(W).astype(np.float64) @ np.abs(X.cpu().numpy()).astype(np.float64))
    assert (np.abs(Y[0].cpu().numpy() - ref) <= bound).all()
