"""LSE of rows with logits far from zero (GPU), whole rows of them and masks beside ordinary
logits, against the float64 sum relative to the row's maximum."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

DEV = "cuda"
F32_MIN = float(np.finfo(np.float32).min)


def _f64(x, T):
    x = x.double().numpy()
    mx = x.max(-1, keepdims=True)
    return (mx[..., 0] / T + np.log(np.exp((x - mx) / T).sum(-1)))


# +-7.4e8: either side of the size (2^30 / log2 e at T = 1) beyond which a row is read again
@pytest.mark.parametrize("value", [-7.4e8, -7.5e8, 7.4e8, 7.5e8, 1e38, -1e9, -1e10, -1e20, -6.9e29, -7e29, -1e31,
                                   -3e38, F32_MIN])
@pytest.mark.parametrize("V", [5, 300, 20001])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("mode", ["het", "mpfr"])
def test_far_rows(mode, dtype, V, value):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    if dtype == "bf16" and value == F32_MIN:
        value = float(torch.finfo(torch.bfloat16).min)
    B, K, gamma = 4, 2, 2
    x = torch.full((B, K, gamma, V), value, dtype=td)
    x[1, :, :, ::2] = float("-inf")   # half of the row masked
    if value < 0:
        x[2, 0, 0, V // 2] = 1.0      # one ordinary logit
        x[3, :, :, 1:V // 2 + 1] = torch.randn(V // 2, generator=torch.Generator().manual_seed(V)).to(td)
    dev = x.to(DEV)
    for T in (0.5, 1.0, 2.0):
        params = psd.make_params(11, V, K, 2, T, T, dtype=td, mode=psd.PSD_MODE_MPFR if mode == "mpfr" else psd.PSD_MODE_HET)
        ws = psd.new_workspace(params, B, gamma, DEV)
        toks = torch.empty((B, K, gamma), dtype=torch.int32, device=DEV)
        lse = torch.empty((B, K, gamma), dtype=torch.float32, device=DEV)
        psd.draft(params, ws, torch.zeros((B, 2), dtype=torch.int32, device=DEV),
                  torch.arange(B, dtype=torch.int64, device=DEV), gamma, 0, dev, toks, lse)
        torch.cuda.synchronize()
        assert psd.workspace_errors(ws) == 0
        want, got = _f64(x.float(), T), lse.cpu().double().numpy()
        far = np.abs(want) > float(np.finfo(np.float32).max)  # (the LSE itself overflows float32)
        assert (got[far] == np.sign(want[far]) * np.inf).all()
        # |row maximum / T| is rounded a few times in float32; its other terms add at most ln V
        assert np.allclose(got[~far], want[~far], rtol=1e-6, atol=1e-5), (T, got, want)
        assert (toks >= 0).all() and (toks.cpu()[1] % 2 == 1).all()
