"""GPU parity of the device front-end (uniform quantizer of Section V-B, device-side CER / CSER
encoder) against the CPU oracle, through the C ABI.  Everything here is integer / byte work, so the
bar is bit-exact: codes, codebook bit patterns, and every array of the encoded handle."""
import numpy as np
import pytest

import oracle
from oracle import quantizer as oq
from paper_1805_10692_amd import binding as B
from paper_1805_10692_amd import workloads as wl
from test_host_library import _compare

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-5


def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: GPU parity tests need a real MI355X")
    return torch.device("cuda:0")


def _to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(_gpu())


def _check_product(h, fmt, W, X):
    """The product of a device-encoded handle at the case's batch and, where that is wider, at batch 1 as well (the
    batch-1 kernel reads the rank table that the device-side encoder derives for the handle)."""
    for Xb in ([X] if X.shape[1] == 1 else [X, np.ascontiguousarray(X[:, :1])]):
        A_scale = oracle.abs_dot_dense(W, Xb, threads=8)
        want = oracle.dot_dense(W, Xb, threads=8)
        Yd = torch.full((W.shape[0], Xb.shape[1]), float("nan"), dtype=torch.float32, device=_gpu())
        (B.cer_matmul if fmt == "cer" else B.cser_matmul)(h, _to_dev(Xb), Yd, Xb.shape[1])
        torch.cuda.synchronize()
        Y = Yd.cpu().numpy().astype(np.float64)
        assert np.isfinite(Y).all()
        assert np.all(np.abs(Y - want) <= TOL * A_scale)


ENCODE_CASES = {
    "c1": lambda: wl.config1(),
    "alexnet_s8": lambda: wl.alexnet_fc6(L=2, scale=8),
    "vgg_s8": lambda: wl.vgg_fc6(L=1, scale=8),
    "sweep_K256_p99": lambda: wl.sweep_cell(256, 0.99, L=3, scale=4),
    "sweep_K256_p50": lambda: wl.sweep_cell(256, 0.5, L=3, scale=4),
    "sweep_K2_p70": lambda: wl.sweep_cell(2, 0.7, L=3, scale=4),
    "conv_s4": lambda: wl.conv3x3(L=5, scale=4),
    "conv_s4_dom": lambda: wl.conv3x3(L=5, nonzero_dominant=True, scale=4),
    "u8_index": lambda: wl.random_lowentropy(m=70, n=250, K=6, p_dom=0.6, L=1, seed=31),
    "u32_index": lambda: wl.random_lowentropy(m=9, n=70001, K=8, p_dom=0.9, L=2, seed=33),
    "one_row": lambda: wl.random_lowentropy(m=1, n=3000, K=16, p_dom=0.7, L=1, seed=36),
    "one_col": lambda: wl.random_lowentropy(m=300, n=1, K=3, p_dom=0.5, L=4, seed=37),
    "constant": lambda: wl.random_lowentropy(m=10, n=100, K=1, p_dom=1.0, L=3, seed=38),
    "ragged_63": lambda: wl.random_lowentropy(m=131, n=63, K=9, p_dom=0.4, L=2, seed=41),
    "ragged_65": lambda: wl.random_lowentropy(m=5, n=65, K=200, p_dom=0.2, L=2, seed=42, ratio=0.99),
    "K256_flat": lambda: wl.random_lowentropy(m=37, n=1999, K=256, p_dom=0.05, L=2, seed=43, ratio=0.999),
}


@pytest.mark.parametrize("fmt", ["cer", "cser"])
@pytest.mark.parametrize("name", list(ENCODE_CASES))
def test_encode_device_matches_oracle(name, fmt):
    w = ENCODE_CASES[name]()
    print(f"case {w.name} {fmt} m={w.m} n={w.n}", flush=True)
    A = oracle.encode(w.W, w.codebook, fmt)
    h = B.cer_encode_device(_to_dev(w.W), w.m, w.n, w.codebook, fmt)
    _compare(h, A)
    assert np.array_equal((B.cer_decode if fmt == "cer" else B.cser_decode)(h).view(np.uint32),
                          (w.W + np.float32(0)).view(np.uint32))
    _check_product(h, fmt, w.W, w.X)
    B.cer_free(h)


def test_encode_device_rows_without_entries_and_ties():
    """Rows that hold only the most frequent value, a row whose single entry has the highest rank
    (CER pads it with repeated pointers), and two values with equal counts (codebook order decides)."""
    cb = np.array([5.0, 0.0, -1.0, 2.0, 7.0], np.float32)
    W = np.zeros((9, 130), np.float32)
    W[1, 3] = 7.0
    W[1, 100] = 7.0
    W[4, ::2] = -1.0
    W[4, 1::2] = 2.0        # -1 and 2 occur 65 times each: -1 comes first (lower codebook position)
    W[7, 129] = 5.0
    W[8, 0] = 5.0
    for fmt in ("cer", "cser"):
        A = oracle.encode(W, cb, fmt)
        assert A.omega.tolist() == [0.0, -1.0, 2.0, 5.0, 7.0]   # 5 and 7 tie as well: 5 is earlier in the codebook
        h = B.cer_encode_device(_to_dev(W), 9, 130, cb, fmt)
        _compare(h, A)
        B.cer_free(h)


@pytest.mark.parametrize("bits", [1, 2, 4, 7, 8])
@pytest.mark.parametrize("shape", [(37, 1000), (3, 4097), (1, 5), (64, 4096)])
def test_quantizer_codes_bit_exact(shape, bits):
    W = wl.dense_weights(*shape, seed=50 + bits)
    codes, cb = oq.uniform_quantize(W, bits)
    Wd = _to_dev(W)
    cd = torch.full((W.size,), 255, dtype=torch.uint8, device=_gpu())
    Wq = torch.full((W.size,), float("nan"), dtype=torch.float32, device=_gpu())
    got_cb = B.cer_quantize_uniform(Wd, W.size, bits, cd, Wq)
    torch.cuda.synchronize()
    assert got_cb.tobytes() == cb.tobytes()
    assert np.array_equal(cd.cpu().numpy().astype(np.int64), codes.reshape(-1))
    assert Wq.cpu().numpy().tobytes() == cb[codes].reshape(-1).tobytes()


def test_quantizer_ties_and_exact_grid():
    """The hand-checkable grid of the oracle's pin: range [0, 7], 3 bits, halves go to the even code."""
    w = np.array([0.0, 7.0, 0.49, 0.5, 0.51, 1.5, 2.5, 3.5, 2.49, 6.5, 6.51, 5.5, 4.5, 3.0, 1.0, 6.99], np.float32)
    cd = torch.zeros(w.size, dtype=torch.uint8, device=_gpu())
    cb = B.cer_quantize_uniform(_to_dev(w), w.size, 3, cd)
    assert cb.tolist() == [0, 1, 2, 3, 4, 5, 6, 7]
    assert cd.cpu().tolist() == [0, 7, 0, 0, 1, 2, 2, 4, 2, 6, 7, 6, 4, 3, 1, 7]
    assert cd.cpu().tolist() == oq.uniform_quantize(w, 3)[0].tolist()


@pytest.mark.parametrize("fmt", ["cer", "cser"])
@pytest.mark.parametrize("shape,bits", [((64, 1152), 7), ((131, 777), 4), ((40, 300), 8), ((12, 70000), 5), ((5, 200), 1)])
def test_quantize_encode_device_matches_oracle(shape, bits, fmt):
    W = wl.dense_weights(*shape, seed=60 + bits)
    codes, cb = oq.uniform_quantize(W, bits)
    Wq = cb[codes]
    A = oracle.encode(Wq, cb, fmt)
    h, got_cb = B.cer_quantize_encode_device(_to_dev(W), shape[0], shape[1], bits, fmt)
    assert got_cb.tobytes() == cb.tobytes()
    _compare(h, A)
    X = wl.sample_X(np.random.Generator(np.random.PCG64(7)), shape[1], 3)
    _check_product(h, fmt, Wq, X)
    B.cer_free(h)


def test_front_end_degenerate_and_errors():
    dev = _gpu()
    # constant matrix: one point, no indices
    W = np.full((6, 50), 0.125, np.float32)
    h, cb = B.cer_quantize_encode_device(_to_dev(W), 6, 50, 7, "cer")
    assert cb.tolist() == [0.125]
    d = B.cer_get_dims(h)
    assert (d["K"], d["nnz"], d["groups"]) == (1, 0, 0)
    _check_product(h, "cer", W, np.ones((50, 2), np.float32))
    B.cer_free(h)
    # empty matrices go through without touching the device arrays
    h = B.cer_encode_device(None, 0, 17, np.array([0.0, 1.0], np.float32), "cser")
    assert B.cer_get_dims(h)["nnz"] == 0
    B.cer_free(h)
    # error codes
    Wd = _to_dev(np.array([[0.0, 1.0, 3.0]], np.float32))
    with pytest.raises(B.CerError) as e:
        B.cer_encode_device(Wd, 1, 3, np.array([0.0, 1.0], np.float32))
    assert e.value.code == B.CER_E_NOT_IN_CODEBOOK
    with pytest.raises(B.CerError) as e:
        B.cer_encode_device(Wd, 1, 3, np.array([0.0, 1.0, 1.0, 3.0], np.float32))
    assert e.value.code == B.CER_E_BAD_CODEBOOK
    with pytest.raises(B.CerError) as e:
        B.cer_encode_device(Wd, 1, 3, np.arange(300, dtype=np.float32))
    assert e.value.code == B.CER_E_TOO_LARGE
    bad = _to_dev(np.array([[0.0, np.nan, 3.0]], np.float32))
    with pytest.raises(B.CerError) as e:
        B.cer_quantize_encode_device(bad, 1, 3, 4)
    assert e.value.code == B.CER_E_INVALID
    with pytest.raises(B.CerError) as e:
        B.cer_quantize_uniform(bad, 3, 4)
    assert e.value.code == B.CER_E_INVALID
    narrow = _to_dev(np.array([[1.0, 1.0 + 8 * 2.0 ** -23]], np.float32))
    with pytest.raises(B.CerError) as e:
        B.cer_quantize_encode_device(narrow, 1, 2, 8)
    assert e.value.code == B.CER_E_BAD_CODEBOOK
    with pytest.raises(B.CerError) as e:
        B.cer_quantize_uniform(Wd, 3, 9)
    assert e.value.code == B.CER_E_INVALID
    del dev


def test_full_size_vgg_fc6_encode_device():
    """The headline matrix (4096 x 25088, 16 values) converted on the device: every array equals the oracle's."""
    w = wl.vgg_fc6(L=1)
    Wd = _to_dev(w.W)
    for fmt in ("cer", "cser"):
        print(f"full-size encode {fmt}", flush=True)
        A = oracle.encode(w.W, w.codebook, fmt)
        h = B.cer_encode_device(Wd, w.m, w.n, w.codebook, fmt)
        _compare(h, A)
        B.cer_free(h)


def test_full_size_alexnet_fc6_quantize_encode_device():
    """An unquantized 4096 x 9216 layer through the 7-bit quantizer and into CER, all on the device."""
    W = wl.dense_weights(4096, 9216, seed=9)
    codes, cb = oq.uniform_quantize(W, 7)
    A = oracle.encode(cb[codes], cb, "cer")
    h, got_cb = B.cer_quantize_encode_device(_to_dev(W), 4096, 9216, 7, "cer")
    assert got_cb.tobytes() == cb.tobytes()
    _compare(h, A)
    B.cer_free(h)


DECODE_CASES = dict(ENCODE_CASES)
DECODE_CASES["many_groups_u16_ranks"] = lambda: wl.random_lowentropy(m=40, n=9000, K=700, p_dom=0.3, L=1, seed=39, ratio=0.995)
DECODE_CASES["wide_rows_many_groups"] = lambda: wl.random_lowentropy(m=6, n=20003, K=1500, p_dom=0.3, L=1, seed=47, ratio=0.9995)
DECODE_CASES["wide_rows_aligned"] = lambda: wl.random_lowentropy(m=5, n=12288, K=40, p_dom=0.8, L=1, seed=48)
DECODE_CASES["dominant_nonzero"] = lambda: wl.random_lowentropy(m=33, n=500, K=7, p_dom=0.5, L=1, seed=46, dominant=0)


@pytest.mark.parametrize("fmt", ["cer", "cser"])
@pytest.mark.parametrize("name", list(DECODE_CASES))
def test_decode_device_round_trip(name, fmt):
    """Host-encoded handle -> dense matrix on the device: bit for bit the encoder's input (Section III-A)."""
    w = DECODE_CASES[name]()
    h = (B.cer_encode if fmt == "cer" else B.cser_encode)(w.W, w.codebook)
    out = torch.full((w.m, w.n), float("nan"), dtype=torch.float32, device=_gpu())
    B.cer_decode_device(h, out)
    torch.cuda.synchronize()
    B.cer_free(h)
    want = oracle.decode(oracle.encode(w.W, w.codebook, fmt))
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert np.array_equal(want.view(np.uint32), (w.W + np.float32(0)).view(np.uint32))


def test_decode_device_full_size_vgg_fc6():
    """The 4096 x 25088 matrix of the headline workload, decoded on the device, equals the encoder's input."""
    dev = _gpu()
    w = wl.vgg_fc6(L=1)
    Wd = torch.from_numpy(w.W).to(dev)
    for fmt in ("cer", "cser"):
        print(f"full-size decode {fmt}", flush=True)
        h = (B.cer_encode if fmt == "cer" else B.cser_encode)(w.W, w.codebook)
        out = torch.full_like(Wd, float("nan"))
        B.cer_decode_device(h, out)
        torch.cuda.synchronize()
        B.cer_free(h)
        assert torch.equal(out.view(torch.int32), (Wd + 0.0).view(torch.int32))


def test_device_only_round_trip_full_size():
    """Unquantized 4096 x 9216 layer -> quantize + encode -> decode, never leaving the device: the decoded
    matrix equals the quantizer's own output (cer_quantize_uniform's Wq) and the oracle's, bit for bit."""
    dev = _gpu()
    W = wl.dense_weights(4096, 9216, seed=9)
    Wd = torch.from_numpy(W).to(dev)
    Wq = torch.empty_like(Wd)
    cb = B.cer_quantize_uniform(Wd, W.size, 7, None, Wq)
    for fmt in ("cer", "cser"):
        h, cb2 = B.cer_quantize_encode_device(Wd, 4096, 9216, 7, fmt)
        assert cb2.tobytes() == cb.tobytes()
        out = torch.full_like(Wd, float("nan"))
        B.cer_decode_device(h, out)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), (Wq + 0.0).view(torch.int32))
        B.cer_free(h)
    codes, ocb = oq.uniform_quantize(W, 7)
    assert np.array_equal(Wq.cpu().numpy().view(np.uint32), ocb[codes].view(np.uint32))


def test_device_encoded_handle_clones_and_inspects_lazily():
    """A handle encoded on the device has no host copy of its arrays until asked: cloning it, inspecting it,
    pricing it and decoding it on the host must all fetch them and agree with a host-encoded handle."""
    dev = _gpu()
    w = wl.vgg_fc6(L=3, scale=8)
    Wd = _to_dev(w.W)
    for fmt in ("cer", "cser"):
        A = oracle.encode(w.W, w.codebook, fmt)
        hd = B.cer_encode_device(Wd, w.m, w.n, w.codebook, fmt)
        hh = (B.cer_encode if fmt == "cer" else B.cser_encode)(w.W, w.codebook)
        assert B.cer_storage_bits(hd) == B.cer_storage_bits(hh) == oracle.storage_bits(A)     # needs no arrays
        assert B.cer_cost_model(hd) == B.cer_cost_model(hh)                                    # fetches them
        assert B.cer_cost_model(hd, B.CER_COUNT_EXAMPLE) == B.cer_cost_model(hh, B.CER_COUNT_EXAMPLE)
        hc = B.cer_clone_device(hd)
        B.cer_free(hd)                                                                         # the clone stands alone
        _compare(hc, A)
        _check_product(hc, fmt, w.W, w.X)
        assert np.array_equal((B.cer_decode if fmt == "cer" else B.cser_decode)(hc).view(np.uint32), w.W.view(np.uint32))
        B.cer_free(hc)
        B.cer_free(hh)
    del dev


@pytest.mark.parametrize("fmt", ["cer", "cser"])
def test_sizes_of_every_row_reach_the_scan(fmt):
    """Row counts around the sixteen rows of a workgroup and the 4096 rows of a round of the scan, one after the other in the same
    temporary: sizes that another workgroup's scan did not see would be those of the matrix before."""
    _gpu()
    rng = np.random.default_rng(11)
    cb = np.array([0.0, 1.0, -1.0, 0.5, 2.0], np.float32)
    for m in (5003, 1, 15, 4097, 16, 17, 4096, 33, 9000, 4111):
        p0 = rng.uniform(0.3, 0.95)
        W = rng.choice(cb, size=(m, 96), p=[p0] + [(1 - p0) / 4] * 4).astype(np.float32)
        hd = B.cer_encode_device(_to_dev(W), m, 96, cb, fmt)
        hh = (B.cer_encode if fmt == "cer" else B.cser_encode)(W, cb)
        for which in (B.CER_ARRAY_ROWPTR, B.CER_ARRAY_OMEGAPTR, B.CER_ARRAY_COLI, B.CER_ARRAY_OMEGAI):
            assert np.array_equal(B.cer_get_array(hd, which), B.cer_get_array(hh, which)), (m, which)
        B.cer_free(hd)
        B.cer_free(hh)


@pytest.mark.parametrize("at", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", [(1, 3), (5, 4), (7, 1021), (3, 1025), (6, 2050), (5, 4100), (2100, 1030)])
def test_codes_of_rows_at_any_address(shape, at):
    """Rows that begin at any multiple of four bytes, codes at any byte; what lies around the outputs stays as it is.  Most elements
    share three values (the copies of the histogram)."""
    m, n = shape
    W = wl.dense_weights(m, n, seed=n + at)
    W[:, n // 3:] = W[:, :1]
    codes, cb = oq.uniform_quantize(W, 7)
    wb = torch.full((W.size + 4,), 1e30, dtype=torch.float32, device=_gpu())
    wb[at:at + W.size] = _to_dev(W).reshape(-1)
    cd = torch.full((W.size + 4,), 255, dtype=torch.uint8, device=_gpu())
    qb = torch.full((W.size + 4,), 7.5, dtype=torch.float32, device=_gpu())
    Wd, first = wb[at:at + W.size], at ^ 1
    assert B.cer_quantize_uniform(Wd, W.size, 7, cd[first:first + W.size], qb[at:at + W.size]).tobytes() == cb.tobytes()
    torch.cuda.synchronize()
    assert np.array_equal(cd[first:first + W.size].cpu().numpy(), codes.reshape(-1))
    assert qb[at:at + W.size].cpu().numpy().tobytes() == cb[codes].reshape(-1).tobytes()
    assert (cd[:first] == 255).all() and (cd[first + W.size:] == 255).all() and (qb[:at] == 7.5).all() and (qb[at + W.size:] == 7.5).all()
    for fmt in ("cer", "cser"):
        h, _ = B.cer_quantize_encode_device(Wd, m, n, 7, fmt)
        _compare(h, oracle.encode(cb[codes], cb, fmt))
        B.cer_free(h)
