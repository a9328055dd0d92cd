"""Lists raced in float32 first (GPU): enough races that several have runners-up within
the float32 margin and go to the exact code (about one in a thousand has), every form
of the candidates (one per thread up to 256, more, fewer groups than top_k, more than
1024 groups), +inf logits, against the oracle."""
import dataclasses
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import workloads  # noqa: E402
from test_gpu_topk import run_gpu, run_topk  # noqa: E402


@pytest.fixture(scope="module")
def psd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd as m
    return m


@pytest.mark.parametrize("mpfr", [False, True])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("V,K,gamma,B,top_k,dtype", [
    (300, 8, 8, 64, 20, "fp32"),     # 5200 races
    (9000, 4, 3, 16, 64, "bf16"), (9000, 4, 3, 16, 65, "fp32"),  # one group per lane or more than one
    (40000, 3, 2, 8, 256, "bf16"),   # many ties at the cut: more than 256 candidates
    (140000, 2, 2, 4, 50, "bf16"),   # more than 1024 groups
    (200, 32, 2, 8, 200, "fp32")])
def test_lists_against_oracle(psd, V, K, gamma, B, top_k, dtype, layout, mpfr):
    w = workloads.custom(V, K, gamma, B, dtype=dtype, sigma=1.0, alpha=0.5, tau=0.4, cid=960 + K)
    run_topk(psd, w, 3, layout, mpfr, top_k)


@pytest.mark.parametrize("mpfr", [False, True])
@pytest.mark.parametrize("target_rows", [1, 3])
def test_infinite_logit_wins(psd, mpfr, target_rows):
    w = workloads.custom(5000, 3, 2, 2, dtype="fp32", cid=970)
    blk = workloads.make_block(w, seed=9, target_rows=target_rows)
    blk["target_logits"][..., 4321] = np.inf
    blk["draft_logits"][..., 1234] = np.inf
    g = run_gpu(psd, w, blk, 0, mpfr, 50, 1.0, target_rows=target_rows)
    out = g[0] if isinstance(g, tuple) else g
    assert (out["target_tokens"] == 4321).all()
    first = out["draft_tokens"][:, 0, 0]  # (an identical drafter's further samples are other arrivals of it)
    assert (first == 1234).all()


@pytest.mark.parametrize("mpfr", [False, True])
@pytest.mark.parametrize("target_rows", [1, 3])
@pytest.mark.parametrize("T", [1.1754944e-38, 2.9e-39, 1e-39, 1e-45])
def test_temperatures_near_zero(psd, mpfr, target_rows, T):
    """Down to temperatures whose float32 reciprocal overflows, the largest logit wins
    (a scaled difference beyond every clock), and an empty row gives -1."""
    w = dataclasses.replace(workloads.custom(5000, 3, 2, 2, dtype="fp32", cid=971), T_target=T, T_draft=T)
    blk = workloads.make_block(w, seed=9, target_rows=target_rows)
    blk["draft_logits"][1, :, 1] = -np.inf
    g = run_gpu(psd, w, blk, 0, mpfr, 50, 1.0, target_rows=target_rows)
    want = blk["target_logits"].argmax(-1).numpy()
    assert (g["target_tokens"].cpu().numpy() == want).all()
    d, wd = g["draft_tokens"].cpu().numpy(), blk["draft_logits"].argmax(-1).numpy()
    wd[1, :, 1] = -1
    if mpfr:  # (every sample of a context is an arrival of its row's largest token: the paths stay together)
        wd = np.repeat(wd[:, :1], 3, 1)
    assert (d == wd).all()


@pytest.mark.parametrize("top_p", [1.0, 0.9, 0.5, 0.3])
def test_infinite_logits_share_the_mass(psd, top_p):
    """Two +inf logits have probability 1/2 each, every other token 0."""
    w = workloads.custom(5000, 3, 2, 64, dtype="fp32", cid=972)
    blk = workloads.make_block(w, seed=9)
    for t in ("target_logits", "draft_logits"):
        blk[t][..., 17] = blk[t][..., 4321] = np.inf
    g = run_gpu(psd, w, blk, 0, False, 50, top_p)
    # (the exact race of equal infinite scores goes to the lowest token)
    assert (g["target_tokens"] == 17).all() and (g["draft_tokens"] == 17).all()
    assert (g["target_lse"] == np.inf).all() and (g["draft_lse"] == np.inf).all()
