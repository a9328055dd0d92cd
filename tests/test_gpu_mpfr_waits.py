"""Waits between the launches of an identical-drafter call (GPU).

A sampling launch of every depth runs beside the launch that streams the draft rows.  It
must give the right drafts in whatever order the two are dispatched: a sampler whose row
has not come within its polls reads the row itself.  With a spin limit of one poll (set
from the host) that happens for practically every row; with one drafter no draft is
waited for, so the drafts are those of an undisturbed call, bit for bit.
"""
import os
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import workloads  # noqa: E402
from test_gpu_mpfr import run_mpfr  # noqa: E402

DEV = "cuda"


@pytest.fixture(scope="module")
def psd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd as m
    return m


@pytest.mark.parametrize("V,gamma,B,dtype,layout", [
    (128256, 4, 16, "bf16", 0), (50257, 3, 8, "fp32", 0), (700, 8, 64, "bf16", 1), (5, 2, 3, "fp32", 0)])
def test_rows_that_do_not_come_are_read(psd, V, gamma, B, dtype, layout):
    w = workloads.custom(V, 1, gamma, B, dtype=dtype, cid=980)
    blk = workloads.make_block(w, seed=V, device=DEV)
    blk["draft_logits"][0, 0, gamma - 1, :] = float("-inf")  # a row without a finite logit
    ref, _ = run_mpfr(psd, w, 0, layout, blk=blk)
    params = psd.make_params(w.key, V, 1, w.m, w.T_target, w.T_draft, dtype=w.torch_dtype, clocks=layout,
                             mode=psd.PSD_MODE_MPFR)
    ws = psd.new_workspace(params, B, gamma, DEV)
    try:
        psd.set_spin_limit(1)
        out = psd.verify(params, ws, blk["prefix_tokens"], blk["start_pos"], blk["target_logits"],
                         blk["draft_logits"])
        torch.cuda.synchronize()
    finally:
        psd.set_spin_limit(0)
    # (the target race's own waits give up as well: only the drafts are compared)
    assert torch.equal(out["draft_tokens"], ref["draft_tokens"])


@pytest.mark.parametrize("K,B,gamma,V", [
    (4, 95, 3, 3000), (4, 96, 3, 3000), (1, 383, 2, 900), (8, 64, 8, 3000), (16, 48, 4, 5000), (3, 256, 4, 3000),
    (12, 64, 3, 20000), (31, 24, 3, 900), (1, 1023, 2, 900)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_blocks_around_the_residency_limits(psd, K, B, gamma, V, dtype):
    """B K around 384 (the most samplers that run beside the streaming and racing
    launches), 768 (the most that are resident by themselves) and 1024."""
    w = workloads.custom(V, K, gamma, B, dtype=dtype, cid=981)
    blk = workloads.make_block(w, seed=B, device=DEV)
    run_mpfr(psd, w, 0, 0, blk=blk, seqs=range(0, B, max(1, B // 6)))
