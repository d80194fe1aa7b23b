"""How kernels are launched -- which variant, how many workgroups, how much LDS: on the CPU, with the HIP runtime of tests/fake_hip.cpp in the
place of the real one (a process of its own for each case)."""
import os
import subprocess
import sys

import pytest

from test_prepare_errors import fake  # noqa: F401  (the library of that runtime)

HERE = os.path.dirname(os.path.abspath(__file__))

# A matrix of m x n elements, `indexed` of them on one of `values` values (a distance of `step` apart, or without a common one), times `batch` columns.
CHILD = """
import ctypes, sys
import numpy as np
from paper_1805_10692_amd import binding as B
fake = ctypes.CDLL(None)
fake.fake_hip_launch.restype = ctypes.c_char_p
m, n, values, batch, path = (int(a) for a in sys.argv[1:6])
indexed, step = float(sys.argv[6]), float(sys.argv[7])
rng = np.random.default_rng(0)
cb = (np.arange(values) - values // 2).astype(np.float32) * np.float32(step) if step else np.append(0.0, rng.standard_normal(values - 1)).astype(np.float32)
W = np.where(rng.random((m, n)) < indexed, rng.choice(cb[cb != 0], size=(m, n)), 0).astype(np.float32)
h = B.cer_encode(W, cb)
X, Y = np.zeros(n * batch + 4, np.float32), np.zeros(m * batch, np.float32)
opts = B.MatmulOpts(path=path)
at = X.ctypes.data + (-X.ctypes.data) % 16
assert B.lib().cer_matmul_ex(ctypes.c_void_p(h.ptr) if isinstance(h.ptr, int) else h.ptr, ctypes.c_void_p(at), ctypes.c_void_p(Y.ctypes.data), batch, None, ctypes.byref(opts)) == 0
for text in sys.argv[8:]:
    shape = (ctypes.c_uint * 5)()
    name = fake.fake_hip_launch(text.encode(), shape)
    print((name or b"-").decode(), *shape)
"""


def launches(lib, m, n, values, batch, path, indexed, step, *texts):
    env = dict(os.environ, LD_PRELOAD=lib, PYTHONPATH=os.path.dirname(HERE))
    out = subprocess.run([sys.executable, "-c", CHILD, *map(str, (m, n, values, batch, path, indexed, step)), *texts], env=env,
                         capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    return [(line.split()[0], [int(x) for x in line.split()[1:]]) for line in out.stdout.splitlines()]


DENSE = 3


# One segment of n columns rounded up to 32 holds the codes, but a row is written, and its codes are read, up to a multiple of 128 columns: the last
# row's behind all others.
@pytest.mark.parametrize("m,n,step", [(2048, 289, 0.0), (2048, 257, 0.0625), (2048, 384, 0.0), (1024, 7000, 0.0625), (1300, 13000, 0.0625)])
def test_decoder_reads_no_codes_behind_its_memory(fake, m, n, step):  # noqa: F811
    (name, (gx, gy, _, threads, lds)), = launches(fake, m, n, 24, 1024, DENSE, 0.5, step, "decode_tiles_kernel")
    assert name != "-" and gy == 1
    rows = -(-m // gx)
    assert rows in (2, 4, 8)
    seg, pitch = -(-n // 32) * 32, -(-n // 128) * 128
    assert (rows - 1) * (seg + 8) + max(seg + 8, pitch) <= lds <= rows * (seg + 8) + 128
