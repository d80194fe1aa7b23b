"""The native product calls of the binding: argument forms and errors (the products themselves: the GPU tests)."""
import inspect

import numpy as np
import pytest

from paper_1805_10692_amd import binding as B

CALLS = [B.cer_matmul, B.cser_matmul, B.cer_matmul_noalloc, B.csr_matmul]


class NoHandle:
    ptr = None


@pytest.mark.parametrize("call", CALLS)
def test_signature_and_argument_errors(call):
    assert list(inspect.signature(call).parameters) == ["h", "X", "Y", "batch", "stream"]
    with pytest.raises(B.CerError) as e:
        call(NoHandle(), 16, 16, 1, 0)
    assert e.value.code == B.CER_E_INVALID and call.__name__ in str(e.value)
    with pytest.raises(B.CerError):
        call(h=NoHandle(), X=16, Y=16, batch=1, stream=0)
    for args, kw in (((NoHandle(), 16, 16), {}), ((NoHandle(), 16, 16, 1, 0, 0), {}), ((NoHandle(), 16, 16, 1), {"batch": 1}),
                     ((NoHandle(), 16, 16, 1), {"streams": 0}), ((NoHandle(), 16, 16, 1.5, 0), {})):
        with pytest.raises(TypeError):
            call(*args, **kw)
    with pytest.raises(AttributeError):
        call(object(), 16, 16, 1, 0)
    torch = pytest.importorskip("torch")
    with pytest.raises(ValueError):
        call(NoHandle(), torch.zeros(4), 16, 1, 0)  # host memory


def test_host_only_handle():
    h = B.cer_encode(np.ones((2, 4), np.float32), np.ones(1, np.float32))
    with pytest.raises(B.CerError) as e:
        B.cser_matmul(h, 16, 16, 1, 0)
    assert e.value.code == B.CER_E_FORMAT
