"""Memory of a handle that is compressed on the device (csrc/frontend.hip): it is allocated before the number of groups is known, with room for one
group per value and row.  On the CPU, with the HIP runtime of tests/fake_hip.cpp, which tells the sizes in the kernels' place."""
import json
import os
import subprocess
import sys

from paper_1805_10692_amd import binding as B
from test_prepare_errors import fake  # noqa: F401  (the library of that runtime)

HERE = os.path.dirname(os.path.abspath(__file__))
CHILD = """
import ctypes, json, os, sys
import numpy as np
from paper_1805_10692_amd import binding as B
fake = ctypes.CDLL(None)
fake.fake_hip_bytes.restype = ctypes.c_size_t

def encode(m, n, K, cser):
    cb = np.arange(K, dtype=np.float32)
    out = ctypes.c_void_p()
    rc = B.lib().cer_encode_device(ctypes.c_void_p(4096), m, n, ctypes.c_void_p(cb.ctypes.data), K, cser, None, ctypes.byref(out))
    return rc, B.Handle(out.value, "cser" if cser else "cer") if rc == 0 else None

for m, n, K, cser, sizes, fail in json.load(sys.stdin):
    os.environ["FAKE_HIP_SIZES"], os.environ["FAKE_HIP_FAIL"] = sizes, fail
    B.lib().cer_trim()
    rc, h = encode(m, n, K, cser)
    error = B.lib().cer_last_hip_error() if rc else 0
    held, groups = 0, -1
    if h:
        groups = B.cer_get_dims(h)["groups"]
        B.lib().cer_trim()
        held = fake.fake_hip_bytes()
        B.cer_free(h)
        B.lib().cer_trim()
        held -= fake.fake_hip_bytes()
    os.environ["FAKE_HIP_FAIL"] = ""
    print(held, rc, error, groups, encode(m, n, K, cser)[0], flush=True)
"""


def encode(lib, calls):
    """calls: rows, columns, values, CSER, (longest row, indexed elements, groups, groups of a row at most), what fails -> memory held, code, HIP
    error, groups, the code of the same call afterwards"""
    given = [(m, n, K, cser, ":".join(map(str, (longest | K << 32 | K << 41, nnz, groups, groups, most))), fail)
             for m, n, K, cser, (longest, nnz, groups, most), fail in calls]
    env = dict(os.environ, LD_PRELOAD=lib, PYTHONPATH=os.path.dirname(HERE))
    out = subprocess.run([sys.executable, "-c", CHILD], input=json.dumps(given), env=env, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    return [[int(x) for x in line.split()] for line in out.stdout.splitlines()]


# 64 rows of 3000 indexed elements and 100 of 255 groups: 486 KB, 526 with the room (allocated in steps of 64 KiB); the temporary takes less
def test_a_handle_that_fits_without_the_room(fake):  # noqa: F811
    want = {
        "": (0, 0, 6400, 0),
        "malloc:525000:2": (0, 0, 6400, 0),  # the handle itself fits
        "malloc:480000:2": (B.CER_E_HIP, 2, -1, 0),
        "malloc:480000:100": (B.CER_E_HIP, 100, -1, 0),
    }
    got = encode(fake, [(64, 4096, 256, 0, (3000, 64 * 3000, 6400, 100), fail) for fail in want])
    assert {fail: tuple(g[1:]) for fail, g in zip(want, got)} == want


def block(size):
    """Handles' memory comes in steps of an eighth of its power of two."""
    step = 65536
    while step * 16 <= size:
        step *= 2
    return -(-int(size) // step) * step


# Rows of one group each: next to nothing of the room is used.  Bytes per row: two per index, 4 + 8 of pointers, 1024 of the rank table; room for 255
# groups of four bytes, in CSER one more for the rank.
def test_room_is_at_most_half_of_the_rest(fake):  # noqa: F811
    m, K = 4096, 256
    cases = [(cser, indexed) for cser in (0, 1) for indexed in (300, 500, 750, 1100, 2000)]
    for (cser, indexed), (held, rc, *_) in zip(cases, encode(fake, [(m, 4096, K, c, (i, m * i, m, 1), "") for c, i in cases])):
        assert rc == 0
        exact = 2 * m * indexed + 8192 + (4 + cser) * m + 12 * (m + 1) + 4 * K + 4 * K * m + 256
        assert block(exact) <= held <= block(1.5 * exact + 2048), (cser, indexed)
