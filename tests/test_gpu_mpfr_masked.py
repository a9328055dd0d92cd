"""Identical drafters on masked rows (GPU): a drafter whose grammar or sampler leaves one
stretch of the vocabulary, the other logits at -inf, at the type's lowest value or at a
large negative constant.  Contexts of up to 32 samples, one stretch inside a sixteenth of
the row, against the oracle, with no error bit."""
import os
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import workloads  # noqa: E402
from test_gpu_mpfr import run_mpfr  # noqa: E402


@pytest.fixture(scope="module")
def psd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd as m
    return m


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("K", [2, 16, 17, 32])
@pytest.mark.parametrize("fill", [float("-inf"), -1e4, -1e9, float(torch.finfo(torch.bfloat16).min)])
@pytest.mark.parametrize("dtype,lo,n", [("bf16", 20100, 1700), ("fp32", 3, 40)])
def test_one_stretch_of_the_vocabulary(psd, layout, K, fill, dtype, lo, n):
    w = workloads.custom(32000, K, 2, 2, dtype=dtype, sigma=1.0, alpha=0.5, tau=0.3, cid=1000)
    blk = workloads.make_block(w, seed=K)
    blk["draft_logits"][..., :lo] = fill
    blk["draft_logits"][..., lo + n:] = fill
    run_mpfr(psd, w, K, layout, blk=blk)
