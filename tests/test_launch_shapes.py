"""How kernels are launched -- which variant, how many workgroups, how much LDS: on the CPU, with the HIP runtime of tests/fake_hip.cpp in the
place of the real one (a process of its own for each case)."""
import json
import os
import re
import subprocess
import sys

import numpy as np
import pytest

import test_gpu_densify
import test_gpu_early_sizes
import test_gpu_mfma
import test_gpu_narrow
import test_gpu_shared_rows
from paper_1805_10692_amd import binding as B
from test_prepare_errors import fake  # noqa: F401  (the library of that runtime)

HERE = os.path.dirname(os.path.abspath(__file__))

# The GPU tests' own matrices and some more, one product each: what was launched.
SCRIPT = """
import ctypes, json, sys
import numpy as np
from paper_1805_10692_amd import binding as B
from paper_1805_10692_amd import workloads as wl
import test_gpu_densify, test_gpu_mfma, test_gpu_narrow
fake = ctypes.CDLL(None)
fake.fake_hip_launch.restype = ctypes.c_char_p

def product(W, cb, cser, L, path, *texts):
    h = (B.cser_encode if cser else B.cer_encode)(W, cb)
    X, Y = np.zeros(W.shape[1] * L + 4, np.float32), np.zeros(W.shape[0] * L, np.float32)
    at = X.ctypes.data + (-X.ctypes.data) % 16
    opts = B.MatmulOpts(path=path)
    fake.fake_hip_forget()
    assert B.lib().cer_matmul_ex(h.ptr, ctypes.c_void_p(at), ctypes.c_void_p(Y.ctypes.data), L, None, ctypes.byref(opts)) == 0
    B.cer_free(h)
    out = []
    for text in texts:
        shape = (ctypes.c_uint * 7)()
        out.append(((fake.fake_hip_launch(text.encode(), shape) or b"").decode(), list(shape)))
    return out

kind, cases = json.load(sys.stdin)
for case in cases:
    if kind == "rows":
        m, n, p_dom, K, dominant = case
        w = wl.random_lowentropy(m=m, n=n, K=K, p_dom=p_dom, L=1, seed=m + n, ratio=0.99 if K > 128 else 0.7, **({} if dominant is None else {"dominant": dominant}))
        got = product(w.W, w.codebook, False, 1, -1, "cer_gemv_tab_kernel")
    elif kind == "fused":
        m, n, K, p0, L = case
        rng = np.random.default_rng(0)
        cb = (np.arange(K) - K // 2).astype(np.float32) / np.float32(max(K / 2, 1))
        W = np.where(rng.random((m, n)) > p0, rng.choice(cb[cb != 0], size=(m, n)), 0).astype(np.float32)
        got = product(W, cb, False, L, -1, "cer_fused_kernel")
    elif kind == "narrow":
        (m, n, K, p0, L), zero = case
        W, cb, _ = test_gpu_narrow.matrix(m, n, L, K, p0, zero)
        got = product(W, cb, n % 2 == 1 and zero > 0, L, -1, "cer_narrow_kernel")
    else:
        if kind == "ranks":
            W, cb, cser, _ = test_gpu_mfma.rank_case(*case)
        else:
            (W, cb), cser = test_gpu_densify.eight_rows(*case), case[2] == "any"
        # (the products' kernels, not mfma_sum_kernel)
        got = product(W, cb, cser, case[3], 3, "decode_tiles_kernel", "mfma_product_kernel", "mfma_small_kernel")
    print(json.dumps(got), flush=True)
"""


def products(lib, kind, cases):
    env = dict(os.environ, LD_PRELOAD=lib, PYTHONPATH=os.pathsep.join((os.path.dirname(HERE), HERE)))
    out = subprocess.run([sys.executable, "-c", SCRIPT], input=json.dumps((kind, cases)), env=env, capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr
    return zip(cases, map(json.loads, out.stdout.splitlines()), strict=True)


# One segment of n columns rounded up to 32 holds the codes, but a row is written, and its codes are read, up to a multiple of 128 columns: the last
# row's behind all others.  (m, n, values on a grid or anywhere, batch), rows per workgroup
BEHIND = {(2048, 289, "any", 1200): 8, (2048, 257, "grid", 1200): 8, (2048, 384, "any", 1200): 8, (1024, 7000, "grid", 1200): 4, (1100, 13000, "grid", 1200): 4}


def test_decoder_reads_no_codes_behind_its_memory(fake):  # noqa: F811
    for case, got in products(fake, "eight", list(BEHIND)):
        (_, (gx, gy, _, _, lds, *_)), rows = got[0], BEHIND[case]
        assert gx == -(-case[0] // rows) and gy == 1
        seg, pitch = -(-case[1] // 32) * 32, -(-case[1] // 128) * 128
        assert (rows - 1) * (seg + 8) + max(seg + 8, pitch) <= lds <= rows * (seg + 8) + 128


def test_rows_and_waves_of_batch_1(fake):  # noqa: F811
    """Batch 1: rows per workgroup, waves per row, waves and the reads of X, on both sides of the rule's lines."""
    want = dict(test_gpu_shared_rows.SHAPES)
    for case, [(name, (_, _, _, threads, _, rows, meta))] in products(fake, "rows", list(want)):
        assert threads == 64 * (meta >> 16)
        few = re.search(r"cer_gemv_tab_kernelI[a-z](?:Lb[01]E){4}Lb([01])E", name)[1] == "1"
        assert (rows, 1 << ((meta >> 13) & 7), meta >> 16, few) == want[case], case


def test_columns_and_waves_of_narrow_batches(fake):  # noqa: F811
    want = {(case, zero): w for case, *both in test_gpu_narrow.FEW for zero, w in zip((case[2] // 2, 0), both)}
    for key, [(name, (_, _, _, threads, *_))] in products(fake, "narrow", list(want)):
        got = None
        if name:
            columns, few = re.search(r"cer_narrow_kernelI[a-z]Li(\d)ELb(\d)E", name).groups()
            got = (int(columns), threads // 64, few == "1")
        assert got == want[key], key


def _decoded(got):
    """(rows per workgroup of the decoder, its threads, pieces -- 0: ranks --, whether the product reads ranks, whether its tile is the large one)"""
    (decoder, shape), (large, _), (small, _) = got
    pieces, threads = re.search(r"decode_tiles_kernelI[a-z]+Li(\d)ELj(\d+)E", decoder).groups()
    assert int(threads) == shape[3] and bool(large) != bool(small)
    return shape[0], int(threads), int(pieces), "ELb1E" in (large or small), bool(large)


def test_ranks_or_pieces(fake):  # noqa: F811
    """Products through the decoded matrix: rows of the decoder, ranks or pieces, the tile."""
    want = dict(test_gpu_mfma.RANKS)
    for case, got in products(fake, "ranks", list(want)):
        groups, threads, pieces, by_rank, large = _decoded(got)
        assert (pieces == 0) == by_rank
        rows, *other = want[case]
        assert [groups, threads, by_rank, large] == [-(-case[1] // rows), *other], case


def test_decoder_of_eight_rows(fake):  # noqa: F811
    for case, got in products(fake, "eight", test_gpu_densify.EIGHT_ROWS):
        groups, threads, pieces, by_rank, _ = _decoded(got)
        assert (groups, threads) == (256, 512) and by_rank == (case[3] < 100)
        assert pieces == (0 if by_rank else (2 if case[2] == "grid" else 3))


# The emitter is launched early where the call needs no more than the sizes that are told first: without the others, a call that waits for them finds
# the stream idle and reports it.
EARLY = """
import ctypes, json, os, sys
import numpy as np
from paper_1805_10692_amd import binding as B
for m, n, K, cser, sizes in json.load(sys.stdin):
    os.environ["FAKE_HIP_SIZES"] = sizes
    cb = np.arange(K, dtype=np.float32)
    out = ctypes.c_void_p()
    rc = B.lib().cer_encode_device(ctypes.c_void_p(4096), m, n, ctypes.c_void_p(cb.ctypes.data), K, cser, None, ctypes.byref(out))
    print(rc, B.lib().cer_last_hip_error() if rc else 0)
"""


def test_early_emitter(fake):  # noqa: F811
    calls, want = [], []
    for case, early in test_gpu_early_sizes.CASES:
        m, n, K, _ = case
        W, _, _ = test_gpu_early_sizes.matrix(*case)
        values, counts = np.unique(W, return_counts=True)
        rows = (W != values[np.argmax(counts)]).sum(axis=1)
        for cser in (0, 1):
            calls.append((m, n, K, cser, f"{int(rows.max()) | K << 32 | len(values) << 41}:{int(rows.sum())}"))
            want.append((0, 0) if early[cser] else (B.CER_E_HIP, 719))  # hipErrorLaunchFailure
    env = dict(os.environ, LD_PRELOAD=fake, PYTHONPATH=os.path.dirname(HERE))
    out = subprocess.run([sys.executable, "-c", EARLY], input=json.dumps(calls), env=env, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    got = [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    assert got == want, [c for c, g, w in zip(calls, got, want) if g != w]


# Decode + product in one launch, by turns or fenced: (rows, columns, values, share of zeros, batch) on a uniform grid or of one piece -> (form, rows / 16,
# columns / 16 of a tile, waves, by turns)
TURNS = {(2994, 2804, 36, 0.432, 35): (4, 1, 3, 8, True), (1360, 13925, 12, 0.507, 136): (4, 1, 3, 8, False), (982, 1195, 73, 0.6, 228): (4, 1, 4, 8, True),
         (1319, 9448, 12, 0.763, 160): (4, 1, 4, 8, False), (2697, 3684, 64, 0.487, 25): (1, 1, 2, 16, True), (2047, 2349, 2, 0.733, 122): (1, 1, 4, 8, False)}


def test_turns_of_the_product_in_one_launch(fake):  # noqa: F811
    for case, [(name, _)] in products(fake, "fused", list(TURNS)):
        form, rt, ct, waves, turns = map(int, re.search(r"cer_fused_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d+)ELb(\d)E", name).groups())
        assert (form, rt, ct, waves, turns == 1) == TURNS[case], case
