"""Calls of every kind and of different shapes on one workspace that is never cleared (GPU).

What a call publishes is tagged with an epoch of its own, so no later call, whatever its
layout, can take a tagged word that it did not write for one of its own.  Every call
equals the same call on a fresh workspace.
"""
import os
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import workloads  # noqa: E402

DEV = "cuda"
EPOCH_WORD = 5  # control word: epoch of the last completed call
OUTS = ("out_tokens", "out_len", "draft_tokens", "target_tokens")


@pytest.fixture(scope="module")
def psd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21858_amd import psd as m
    return m


def _align(x):
    return (x + 255) // 256 * 256


def _race_bytes(B, K, gamma, V, bf16):
    """Bytes of the race kernel's workspace, where identical-drafter words and kept lists begin."""
    seg = 16384 if bf16 else 8192
    rows = B * K * (2 * gamma + 1)
    nseg, ng, n3 = -(-V // seg), -(-V // 128), -(-V // 2048)
    o = _align(8192)
    for words in (rows, rows * nseg, rows * ng, rows * n3, rows * nseg, 2 * rows):
        o = _align(o + 8 * words)
    return o


class Call:
    def __init__(self, psd, mode, B, top_k=0, rows="shared", seed=0, V=32000, K=4, gamma=4, dtype="bf16"):
        self.psd, self.name = psd, f"{mode} B={B} top_k={top_k} rows={rows}"
        self.w = w = workloads.custom(V, K, gamma, B, dtype=dtype, cid=990)
        self.tr = K if rows == "paths" else 1
        self.blk = workloads.make_block(w, seed=seed, device=DEV, target_rows=self.tr)
        self.params = psd.make_params(w.key, V, K, w.m, w.T_target, w.T_draft, dtype=w.torch_dtype,
                                      mode=psd.PSD_MODE_MPFR if mode == "mpfr" else psd.PSD_MODE_HET, top_k=top_k)
        self.bytes = psd.workspace_bytes(self.params, B, gamma)
        self.want = self(torch.zeros(self.bytes, dtype=torch.uint8, device=DEV))

    def __call__(self, ws):
        status = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        b = self.blk
        out = self.psd.verify(self.params, ws, b["prefix_tokens"], b["start_pos"], b["target_logits"],
                              b["draft_logits"], target_rows=self.tr, want_targets=True, status=status)
        torch.cuda.synchronize()
        assert int(status[0]) == 0, self.name
        return {k: out[k].cpu() for k in OUTS}

    def check(self, ws, what):
        got = self(ws)
        for k in OUTS:
            assert torch.equal(got[k], self.want[k]), (what, self.name, k)


def _shared(calls):
    return torch.zeros(max(c.bytes for c in calls), dtype=torch.uint8, device=DEV)


def test_distinct_drafters_then_identical_ones(psd):
    """The wider block's race slots lie where the smaller block's streamed words do."""
    wide, small = Call(psd, "het", 32), Call(psd, "mpfr", 4, seed=1)
    for n in range(1, 4):
        ws = _shared([wide, small])
        for _ in range(n):
            wide.check(ws, n)
        for _ in range(n):
            small.check(ws, n)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_every_kind_of_call_in_turn(psd, dtype):
    kinds = [Call(psd, m, B, top_k, rows, seed=B + top_k, V=5000, K=3, gamma=3, dtype=dtype)
             for m in ("het", "mpfr") for B in (2, 24) for top_k in (0, 5) for rows in ("shared", "paths")]
    ws = _shared(kinds)
    gen = torch.Generator().manual_seed(5)
    for turn in range(3):
        for i in torch.randperm(len(kinds), generator=gen).tolist():
            kinds[i].check(ws, turn)


def test_one_epoch_for_every_word_of_a_call(psd):
    """After three calls the epoch is 3, and the words that the last identical-drafter
    call streamed carry it: a word of a call never has the tag of the next one."""
    het, mp = Call(psd, "het", 4), Call(psd, "mpfr", 4, seed=1)
    ws = _shared([het, mp])
    het.check(ws, 0)
    mp.check(ws, 1)
    mp.check(ws, 2)
    assert int(ws[4 * EPOCH_WORD:4 * EPOCH_WORD + 4].view(torch.int32)[0]) == 3
    rows, ng = 4 * 4 * 4, 250
    o = _race_bytes(4, 4, 4, 32000, True)
    tags = ws[o:o + 8 * rows * ng].view(torch.int32).view(rows, ng, 2)[..., 1]
    # (at depth 0 the first path's row serves every path)
    streamed = [r for r in range(rows) if r % 4 != 0 or (r // 4) % 4 == 0]
    assert (tags[streamed] == 3).all()


@pytest.mark.parametrize("mode", ["het", "mpfr"])
@pytest.mark.parametrize("rows,top_k", [("shared", 0), ("paths", 0), ("shared", 7), ("paths", 40)])
@pytest.mark.parametrize("K", [1, 4])
def test_no_word_has_the_tag_of_another_call(psd, mode, rows, top_k, K):
    """After one call on a zeroed workspace, every word that another shape may read as a
    slot has tag 0, that call's own epoch, or a high half that is no epoch (the complement
    of a token or a length)."""
    c = Call(psd, mode, 6, top_k, rows, seed=3, V=5000, K=K, gamma=3)
    ws = torch.zeros(c.bytes, dtype=torch.uint8, device=DEV)
    b = c.blk
    if K == 4:
        c.check(ws, 0)
    else:  # (the targets not asked for: the walk takes them from the workspace)
        out = psd.verify(c.params, ws, b["prefix_tokens"], b["start_pos"], b["target_logits"], b["draft_logits"],
                         target_rows=c.tr)
        assert torch.equal(out["out_tokens"].cpu(), c.want["out_tokens"])
    tags = ws[8192:c.bytes // 8 * 8].view(torch.int32).view(-1, 2)[:, 1].cpu().long() & 0xFFFFFFFF
    epoch = int(ws[4 * EPOCH_WORD:4 * EPOCH_WORD + 4].view(torch.int32)[0])
    other = tags[(tags != 0) & (tags != epoch) & (tags < 0xFFF80000)]
    assert other.numel() == 0, other[:8].tolist()


@pytest.mark.parametrize("mode,top_k", [("het", 0), ("mpfr", 0)])
def test_last_epochs(psd, mode, top_k):
    """The epochs before the last one and after it wrap to 1, never to a kept list's words."""
    c = Call(psd, mode, 2, top_k, seed=4, V=3000, K=2, gamma=2)
    ws = torch.zeros(c.bytes, dtype=torch.uint8, device=DEV)
    word = ws[4 * EPOCH_WORD:4 * EPOCH_WORD + 4].view(torch.int32)
    word.fill_(0xFFF80000 - 2 - (1 << 32))
    for want in (0xFFF80000 - 1, 1, 2):
        c.check(ws, want)
        assert int(word[0]) & 0xFFFFFFFF == want
