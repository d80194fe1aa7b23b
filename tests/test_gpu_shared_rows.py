"""GPU parity of the batch-1 stream kernel on matrices of few rows, where a row is shared by 4 or 8 waves of a
workgroup (each takes a contiguous share of the row's windows, the partial sums meet in LDS): every element against
the oracle's group-sum product (Algorithm 3 / 4), in both formats, with the rows shared (the library's choice) and
whole (CER_OPT_ROWS_WHOLE), which must agree with each other to rounding as well."""
import numpy as np
import pytest

import oracle
from paper_1805_10692_amd import binding as B
from paper_1805_10692_amd import workloads as wl
from test_gpu_parity import check, full_check, run_matmul

pytestmark = pytest.mark.gpu

STREAM = B.MatmulOpts(path=B.CER_PATH_GEMV)
WHOLE = B.MatmulOpts(path=B.CER_PATH_GEMV, flags=B.CER_OPT_ROWS_WHOLE)
# the same kernel finding its group boundaries through rowPtr / OmegaPtr instead of the handle's rank table
NO_TABLE = B.MatmulOpts(path=B.CER_PATH_GEMV, flags=B.CER_OPT_NO_RANK_TABLE)
NO_TABLE_WHOLE = B.MatmulOpts(path=B.CER_PATH_GEMV, flags=B.CER_OPT_NO_RANK_TABLE | B.CER_OPT_ROWS_WHOLE)

CASES = {
    # 16-bit indices: windows of 512 positions
    "one_row_8_windows": lambda: wl.random_lowentropy(m=1, n=20000, K=16, p_dom=0.8, L=1, seed=71),
    "seven_rows_dom": lambda: wl.random_lowentropy(m=7, n=5000, K=5, p_dom=0.4, L=1, seed=72, dominant=4),  # Omega[0] != 0
    "two_windows": lambda: wl.random_lowentropy(m=100, n=1500, K=8, p_dom=0.4, L=1, seed=73),
    "share_ends_on_a_window_edge": lambda: wl.random_lowentropy(m=64, n=4096, K=2, p_dom=0.5, L=1, seed=74),
    "more_waves_than_windows": lambda: wl.random_lowentropy(m=20, n=2500, K=6, p_dom=0.55, L=1, seed=75),
    "many_groups_general_list": lambda: wl.random_lowentropy(m=40, n=9000, K=700, p_dom=0.3, L=1, seed=76, ratio=0.995),
    "eight_rows_per_unit": lambda: wl.random_lowentropy(m=2000, n=3000, K=16, p_dom=0.5, L=1, seed=77),
    "four_rows_per_unit": lambda: wl.random_lowentropy(m=1000, n=6000, K=16, p_dom=0.6, L=1, seed=78),
    "unequal_rows": lambda: _unequal(),
    "lds_edge": lambda: wl.random_lowentropy(m=33, n=38000, K=8, p_dom=0.8, L=1, seed=79),
    # 8-bit indices: windows of 1024 positions, so only a row of 256 columns that is nearly all indexed stays whole
    "u8_index": lambda: wl.random_lowentropy(m=50, n=256, K=6, p_dom=0.05, L=1, seed=80),
}


def _unequal():
    """Rows from empty to completely indexed: shares that are empty, shares behind the row's end."""
    rng = np.random.default_rng(81)
    cb = np.array([0.0, 0.5, -1.0, 2.0, 0.25, -0.125], np.float32)
    W = cb[rng.choice(6, size=(60, 6000), p=[0.6, 0.1, 0.1, 0.1, 0.05, 0.05])].astype(np.float32)
    W[3] = 0.0
    W[4, 1:] = 0.0
    W[5] = cb[rng.integers(1, 6, size=6000)]
    W[6, :700] = 0.0
    W[7, 511:] = 0.0
    W[8, 513:] = 0.0
    X = rng.standard_normal((6000, 1)).astype(np.float32)

    class Case:
        pass
    w = Case()
    w.name, w.W, w.codebook, w.X, w.m, w.n, w.L = "unequal rows", W, cb, X, 60, 6000, 1
    return w


@pytest.mark.parametrize("name", list(CASES))
def test_shared_rows_all_elements(name):
    w = CASES[name]()
    full_check(w, opts=STREAM, want_path=0)
    full_check(w, opts=WHOLE, want_path=0)
    full_check(w, opts=NO_TABLE, want_path=0)
    full_check(w, opts=NO_TABLE_WHOLE, want_path=0)
    scale = oracle.abs_dot_dense(w.W, w.X, threads=8)
    for fmt in ("cer", "cser"):
        a = run_matmul(fmt, w.W, w.codebook, w.X, opts=STREAM)
        b = run_matmul(fmt, w.W, w.codebook, w.X, opts=WHOLE)
        check(a, b.astype(np.float64), 2.0 * scale, f"{name}/{fmt}: shared against whole rows")


@pytest.mark.parametrize("dom", [False, True])
def test_conv3x3_batch1_full_size(dom):
    full_check(wl.conv3x3(L=1, nonzero_dominant=dom))
    full_check(wl.conv3x3(L=1, nonzero_dominant=dom), opts=NO_TABLE)


SHAPES = [  # (m, n, p_dom, K, dominant), (rows, waves per row, waves, whether the reads of X are all on their way) of a workgroup
    ((513, 3300, 0.5, 16, None), (3, 2, 6, True)),              # just above three windows
    ((768, 3801, 0.4, 100, None), (3, 2, 6, True)),             # fewer than five
    ((768, 9001, 0.4, 100, None), (3, 4, 12, False)),           # ten; two tiles of ranks
    ((600, 37000, 0.85, 40, None), (3, 4, 16, False)),          # X and the lists of few waves fill LDS
    ((769, 3001, 0.45, 8, 5), (4, 2, 8, True)),                 # Omega[0] != 0
    ((1024, 12001, 0.5, 4, None), (4, 2, 8, True)),             # fewer than fourteen windows
    ((1024, 16001, 0.5, 4, None), (4, 4, 16, False)),           # fifteen
    ((1025, 9000, 0.5, 16, 3), (5, 2, 10, False)),
    ((1279, 24004, 0.93, 16, None), (5, 1, 16, True)),          # whole rows, X of 96 KB
    ((1300, 5000, 0.3, 64, None), (6, 2, 12, False)),           # seven windows
    ((1300, 5000, 0.55, 64, 7), (4, 1, 4, False)),              # four: whole, an X of 20 KB
    ((1700, 8601, 0.5, 16, 3), (7, 1, 8, True)),                # fewer than nine
    ((1700, 9801, 0.5, 16, 3), (7, 2, 14, False)),
    ((1700, 20001, 0.79, 16, 3), (7, 2, 14, False)),            # more than eight, X of more than 64 KiB
    ((1700, 9801, 0.5, 200, None), (7, 1, 8, True)),            # fewer than 9.8, more than 128 values
    ((1700, 13001, 0.8, 16, None), (7, 1, 8, True)),            # six loads of X for every wave
    ((2048, 7001, 0.5, 5, None), (8, 1, 8, True)),
    ((2048, 9801, 0.5, 5, None), (8, 1, 8, True)),              # fewer than 9.8
    ((2048, 10401, 0.5, 5, None), (8, 2, 16, False)),           # more
    ((2048, 16501, 0.7, 5, None), (8, 2, 16, False)),           # more than 9.5, X of more than 64 KiB
    ((2048, 11301, 0.5, 200, None), (8, 1, 8, True)),           # fewer than 11.5, more than 128 values
    ((2048, 12301, 0.5, 200, None), (8, 2, 16, False)),
    ((500, 2048, 0.7, 9, None), (2, 1, 4, False)),              # two windows
    ((500, 9001, 0.5, 9, None), (2, 4, 8, False)),
    ((2049, 7001, 0.5, 16, 9), (9, 1, 9, False)),               # nine whole rows
    ((2049, 4601, 0.1, 200, None), (9, 1, 9, False)),           # an X of up to 24 KiB, more than 6.5 windows
    ((3072, 5001, 0.1, 200, None), (4, 1, 4, False)),           # twelve rows of an X of up to 24 KiB: workgroups of four waves
    ((3840, 1900, 0.1, 200, None), (4, 1, 4, False)),           # fifteen rows of few windows: the same
    ((3840, 4001, 0.1, 200, None), (4, 1, 4, False)),           # of fewer than 7.5 as well
    ((3840, 5001, 0.1, 200, None), (15, 1, 15, False)),         # of more: one workgroup of as many waves as rows
    ((3840, 6201, 0.5, 5, None), (15, 1, 15, False)),           # an X of more than 24 KiB
]


@pytest.mark.parametrize("m,n,p_dom,K,dominant", [case for case, _ in SHAPES])
def test_waves_per_compute_unit(m, n, p_dom, K, dominant):
    """A workgroup per compute unit of 3 to 15 rows, shared by waves or whole, on both sides of the rule's lines
    (tests/test_launch_shapes.py holds what a workgroup gets against the list)."""
    kw = {} if dominant is None else {"dominant": dominant}
    w = wl.random_lowentropy(m=m, n=n, K=K, p_dom=p_dom, L=1, seed=m + n, ratio=0.99 if K > 128 else 0.7, **kw)  # (every value occurs)
    full_check(w, want_path=0)


def test_few_long_rows_among_short_ones():
    """Rows of unequal length: the longest row alone asks for shares, those of the short rows are empty."""
    rng = np.random.default_rng(5)
    cb = np.array([0.0, 0.5, -1.0, 2.0], np.float32)
    W = cb[rng.choice(4, size=(700, 9000), p=[0.97, 0.01, 0.01, 0.01])].astype(np.float32)
    W[17] = cb[rng.integers(1, 4, size=9000)]
    W[699] = cb[rng.integers(1, 4, size=9000)]
    W[300] = 0.0

    class Case:
        pass
    w = Case()
    w.name, w.W, w.codebook, w.m, w.n, w.L = "few long rows", W, cb, 700, 9000, 1
    w.X = rng.standard_normal((9000, 1)).astype(np.float32)
    full_check(w, want_path=0)
