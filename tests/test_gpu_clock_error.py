"""The float32 clock functions' errors against the float64 ones (GPU): the bounds that the
margins of the float32 decisions rest on."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "_build", "libclock_error.so")


@pytest.fixture(scope="module")
def error():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = ctypes.CDLL(LIB)

    def run(name, *args):
        out = torch.zeros(1, dtype=torch.int32, device="cuda")
        f = getattr(lib, "clock_error_" + name)
        f.argtypes = [ctypes.c_void_p] + [ctypes.c_uint32] * len(args) + [ctypes.c_void_p]
        assert f(out.data_ptr(), *args, torch.cuda.current_stream().cuda_stream) == 0
        e = float(out.cpu().numpy().view(np.float32)[0])
        print(f"[clock error] {name} {args}: {e:.3e}")
        return e

    return run


def test_exp1_of_every_uniform(error):
    assert 0.0 < error("exp1") <= 1.7e-7


def test_ln_of_every_clock_size(error):
    # 4e-6 is what the float32 orders assume.  log2 x is at most 44, where an ulp is 3.8e-6:
    # a hardware error of 1.1 ulp times ln 2 is 2.9e-6, and the product's rounding 0.95e-6
    assert 0.0 < error("ln") <= 4e-6


@pytest.mark.parametrize("V", [7, 1000, 32000, 128256, 1 << 19])
def test_tree_clocks(error, V):
    # at most six rounded terms of 1.7e-7, each with a hardware reciprocal (1.2e-7) and the
    # sum's own rounding
    assert 0.0 < error("tree", V, 5) <= 1e-6
