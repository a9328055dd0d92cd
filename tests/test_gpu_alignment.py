"""Rows at any element boundary (GPU): logits that start off the 16-byte grid, and
vocabularies that are not a multiple of 8, give exactly what an aligned copy gives,
in every path that streams rows (distinct and identical drafters, top-k), and the
oracle's tokens."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import oracle  # noqa: E402
import workloads  # noqa: E402

DEV = "cuda"


@pytest.fixture(scope="module")
def psd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd as m
    return m


def _shifted(t, off):
    """The same values starting `off` elements into a fresh allocation."""
    buf = torch.empty(t.numel() + off, dtype=t.dtype, device=t.device)
    buf[off:] = t.reshape(-1)
    return buf[off:].view(t.shape)


@pytest.mark.parametrize("mode,top_k", [("het", 0), ("mpfr", 0), ("het", 20), ("mpfr", 20)])
@pytest.mark.parametrize("V", [1, 7, 8, 9, 15, 1001, 2049, 16384, 16391, 33003])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_rows_at_any_boundary(psd, dtype, V, mode, top_k):
    w = workloads.custom(V, 3, 2, 3, dtype=dtype, cid=910 + V % 50)
    blk = workloads.make_block(w, seed=V)
    params = psd.make_params(w.key, V, w.K, w.m, w.T_target, w.T_draft, dtype=w.torch_dtype, top_k=top_k,
                             mode=psd.PSD_MODE_MPFR if mode == "mpfr" else psd.PSD_MODE_HET)
    g = {k: v.to(DEV) for k, v in blk.items() if isinstance(v, torch.Tensor)}
    got = []
    for off in (0, 1, 3, 7):  # 0: allocations are 256-byte aligned
        ws = psd.new_workspace(params, w.B, w.gamma, DEV)
        o = psd.verify(params, ws, g["prefix_tokens"], g["start_pos"], _shifted(g["target_logits"], off),
                       _shifted(g["draft_logits"], off), want_lse=True, want_targets=True)
        torch.cuda.synchronize()
        assert psd.workspace_errors(ws) == 0
        got.append({k: v.cpu().numpy() for k, v in o.items()})
    for o in got[1:]:
        for k, v in got[0].items():
            assert np.array_equal(v, o[k]), (k, v, o[k])
    if mode == "het" and not top_k:
        ref = oracle.verify_block(key=w.key, K=w.K, gamma=w.gamma, m=w.m, T_target=w.T_target, T_draft=w.T_draft,
                                  prefix=blk["prefix_tokens"].numpy(), start_pos=blk["start_pos"].numpy(),
                                  target_logits=workloads.as_f32_numpy(blk["target_logits"]),
                                  draft_logits=workloads.as_f32_numpy(blk["draft_logits"]), gpu=got[0])
        assert ref["stats"]["mismatch"] == 0, ref["stats"]["mismatches"]
        for (b, s), v in ref["target_lse"].items():
            assert abs(got[0]["target_lse"][b][s] - v) <= 1e-5 * max(1.0, abs(v))
