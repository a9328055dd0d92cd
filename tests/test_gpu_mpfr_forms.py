"""Every form of an identical-drafter call gives the same drafts (GPU): with and without
the log-sum-exps (rows that only the LSE needs are then not read), fused, drafted depth
by depth, from the fixed scratch and under stream capture, for blocks whose draft rows
stream in one launch (B K < 1024) and in one per depth, and for lists that run full
(equal logits, 32 drafters); the first form is checked against the oracle."""
import os
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import workloads  # noqa: E402
from test_gpu_mpfr import run_mpfr  # noqa: E402

DEV = "cuda"


@pytest.mark.parametrize("V,K,gamma,B,dtype,sigma,layout", [
    (5, 32, 2, 2, "fp32", 0.0, 0), (5, 32, 2, 2, "fp32", 0.0, 1), (129, 32, 2, 2, "bf16", 0.0, 0),
    (4100, 32, 2, 3, "fp32", 0.0, 0), (33001, 16, 3, 4, "bf16", 0.3, 0), (140000, 8, 2, 2, "bf16", 0.0, 0),
    (20000, 5, 3, 40, "fp32", 2.0, 0), (1000, 8, 2, 128, "bf16", 2.0, 0), (4099, 8, 3, 130, "fp32", 1.0, 0),
    (4099, 8, 2, 130, "bf16", 1.0, 1), (7, 32, 2, 33, "bf16", 1.0, 0)])
def test_forms_agree(V, K, gamma, B, dtype, sigma, layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd
    w = workloads.custom(V, K, gamma, B, dtype=dtype, sigma=sigma, alpha=1.0 if sigma else 0.0, tau=sigma * 0.4, cid=950)
    blk = workloads.make_block(w, seed=V + K, device=DEV)
    out, _ = run_mpfr(psd, w, 0, layout, blk=blk, seqs=range(0, B, max(1, B // 4)))
    want = {k: out[k].cpu() for k in ("draft_tokens", "out_tokens", "out_len", "target_tokens")}
    params = psd.make_params(w.key, V, K, w.m, w.T_target, w.T_draft, dtype=w.torch_dtype, clocks=layout,
                             mode=psd.PSD_MODE_MPFR)
    ws = psd.new_workspace(params, B, gamma, DEV)
    args = (blk["prefix_tokens"], blk["start_pos"], blk["target_logits"])
    status = torch.full((1,), -1, dtype=torch.int32, device=DEV)

    def same(o, what):
        torch.cuda.synchronize()
        assert int(status[0]) == 0 and psd.workspace_errors(ws) == 0, what
        for k, v in want.items():
            assert torch.equal(o[k].cpu(), v), (what, k)

    same(psd.verify(params, ws, *args, blk["draft_logits"], want_targets=True, status=status), "tokens only")
    for lse in (None, torch.zeros((B, K, gamma), dtype=torch.float32, device=DEV)):
        dt = torch.full((B, K, gamma), -7, dtype=torch.int32, device=DEV)
        for s in range(gamma):
            psd.draft(params, ws, *args[:2], gamma, s, blk["draft_logits"][:, :, s:s + 1].contiguous(), dt, lse)
        same(psd.verify(params, ws, *args, None, dt, want_targets=True, status=status), "depth by depth")
        if lse is not None:
            assert torch.equal(lse.cpu(), out["draft_lse"].cpu())
    o = psd.verify(params, ws, *args, blk["draft_logits"], want_targets=True, status=status)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o = psd.verify(params, ws, *args, blk["draft_logits"], want_targets=True, status=status, out=o,
                       draft_tokens=o["draft_tokens"])
    for _ in range(3):
        for v in o.values():
            v.zero_()
        graph.replay()
        same(o, "captured")
    try:
        o = psd.verify_static(params, *args, blk["draft_logits"], status=status,
                              out={"target_tokens": torch.zeros_like(want["target_tokens"], device=DEV)})
        same(o, "fixed scratch")
    except psd.PsdError as e:
        assert e.status == psd.PSD_E_WORKSPACE  # the block needs more than the fixed scratch
