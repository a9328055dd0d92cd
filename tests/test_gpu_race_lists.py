"""Races whose work lists run full (GPU): nearly flat rows with many slots list more
level-3 nodes, groups and halves than one pass holds, so the tree descent empties its
lists several times and repeats overflowing passes.  Tokens, tau and LSE against the
oracle, with no error bit."""
import os
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import oracle  # noqa: E402
import workloads  # noqa: E402

DEV = "cuda"


# sigma 0 (and alpha 0): every logit equal, the loosest bounds a row can give
@pytest.mark.parametrize("V,K,sigma", [(1, 32, 0.0), (129, 32, 0.0), (4100, 32, 0.0), (33000, 16, 0.0), (33000, 3, 0.02),
                                       (70001, 32, 0.3), (140000, 8, 0.0), (140000, 8, 1.0)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_full_lists(dtype, V, K, sigma):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd
    w = workloads.custom(V, K, 2, 1, dtype=dtype, sigma=sigma, alpha=0.0, tau=sigma, cid=930 + K)
    blk = workloads.make_block(w, seed=V + K)
    params = psd.make_params(w.key, V, K, w.m, w.T_target, w.T_draft, dtype=w.torch_dtype)
    ws = psd.new_workspace(params, w.B, w.gamma, DEV)
    g = {k: v.to(DEV) for k, v in blk.items() if isinstance(v, torch.Tensor)}
    out = psd.verify(params, ws, g["prefix_tokens"], g["start_pos"], g["target_logits"], g["draft_logits"],
                     want_lse=True, want_targets=True)
    torch.cuda.synchronize()
    assert psd.workspace_errors(ws) == 0
    gpu = {k: v.cpu().numpy() for k, v in out.items()}
    ref = oracle.verify_block(key=w.key, K=K, gamma=w.gamma, m=w.m, T_target=w.T_target, T_draft=w.T_draft,
                              prefix=blk["prefix_tokens"].numpy(), start_pos=blk["start_pos"].numpy(),
                              target_logits=workloads.as_f32_numpy(blk["target_logits"]),
                              draft_logits=workloads.as_f32_numpy(blk["draft_logits"]), gpu=gpu)
    assert ref["stats"]["mismatch"] == 0, ref["stats"]["mismatches"]
    n = int(gpu["out_len"][0])
    assert n == ref["out_len"][0] and list(gpu["out_tokens"][0][:n]) == ref["out_tokens"][0]
    for (b, s), v in ref["target_lse"].items():
        assert abs(gpu["target_lse"][b][s] - v) <= 1e-5 * max(1.0, abs(v))
