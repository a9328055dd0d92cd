"""Races with more near-ties than half the candidate list (GPU).

Logits set to T ln E of the exact clocks tie every chosen token within float32, so the
tree race's list is compacted (a branch with barriers, taken by every thread on one count)
and the float64 decision picks among all of them.
"""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

DEV = "cuda"


# (V, tied tokens): the list holds 256 entries and is compacted above 128; the up to 8
# seed tokens may be listed twice
@pytest.mark.parametrize("V,n_tied", [(129, 129), (200, 200), (4000, 128), (4000, 140), (4000, 240), (130000, 240)])
@pytest.mark.parametrize("layout", [0, 1])
def test_many_near_ties(V, n_tied, layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd
    B, T = 6, 0.75
    params = psd.make_params(77, V, 1, 2, T, T, dtype=torch.float32, clocks=layout)
    gen = torch.Generator().manual_seed(V + n_tied)
    prefix = torch.randint(0, V, (B, 2), generator=gen, dtype=torch.int32).to(DEV)
    start = torch.arange(100, 100 + B, dtype=torch.int64, device=DEV)
    kappa = psd.context_keys(params, start, prefix)
    tokens = torch.stack([torch.randperm(V, generator=gen)[:n_tied].sort().values for _ in range(B)]).to(torch.int32)
    flat = tokens.reshape(-1).to(DEV)
    clocks = psd.clock_values(params, kappa.repeat_interleave(n_tied, 0).contiguous(), torch.zeros_like(flat), flat)
    clocks = clocks.view(B, n_tied).cpu().double().numpy()
    logits = torch.full((B, 2, V), -np.inf)
    for b in range(B):
        logits[b, 0, tokens[b].long()] = torch.from_numpy((T * np.log(clocks[b])).astype(np.float32))
        logits[b, 1, 0] = 0.0
    tied = np.take_along_axis(logits[:, 0].numpy(), tokens.numpy(), 1).astype(np.float64)
    want = np.take_along_axis(tokens.numpy(), np.argmin(np.log(clocks) - tied / float(np.float32(T)), 1)[:, None], 1)[:, 0]
    ws = psd.new_workspace(params, B, 1, DEV)
    g = logits.to(DEV)
    out = psd.verify(params, ws, prefix, start, g, g[:, None, :1].contiguous(), want_targets=True)
    torch.cuda.synchronize()
    assert psd.workspace_errors(ws) == 0
    assert np.array_equal(out["target_tokens"][:, 0].cpu().numpy(), want)
    assert np.array_equal(out["draft_tokens"][:, 0, 0].cpu().numpy(), want)
    assert (out["out_len"].cpu().numpy() == 2).all()
