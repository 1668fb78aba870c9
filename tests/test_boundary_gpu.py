"""Failure handling of prepared drafting calls through the C ABI, by the persistent kernel and by the launches
per position, forced from the host so that every kernel exits normally:

* a workspace whose error word is already set (an earlier stalled hand-off) makes a call write
  token -1 everywhere and NaN statistics, and dls_draft_block_error reports the word; a
  zero-filled workspace works again;
* a prepared buffer that belongs to another head (same shapes, other tensors) is refused by
  the kernels (DLS_DRAFT_ERR_PREPARED) with the same sentinels; the error word is sticky;
* no route leaves words in a workspace that another one could take for its own.
"""
import numpy as np
import pytest
import torch

from paper_2607_07409_amd import binding as B
from paper_2607_07409_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [dict(V=5003, d=96, H=128, r=128, B=7, batch=3),      # persistent kernel, narrow
          dict(V=4099, d=128, H=128, r=128, B=5, batch=37),    # launches per position
          dict(V=4099, d=128, H=128, r=128, B=5, batch=11)]    # persistent kernel, wide


def _setup(i, seed=None):
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(dtype="bf16", **SHAPES[i])
    hw = W.make_head(wl, "stress", seed=seed)
    head = B.LocalHead.from_weights(hw).prepare()
    lt = B.as_tensor(W.make_long_logits(wl))
    last = torch.from_numpy(W.make_last_token(wl)).cuda()
    assert head.path(wl.batch, wl.B, lt.dtype, False) == 1
    return wl, head, lt, last


def _call(head, lt, last, ws):
    tok, st = B.draft_block(head, lt, last, None, 1.0, 0.5, 0.0, workspace=ws, exclusive_device=False)
    torch.cuda.synchronize()
    return tok, st


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_preset_error_word_gives_sentinels(i):
    wl, head, lt, last = _setup(i)
    ws = B.draft_workspace(head, wl.batch, wl.B)
    good_tok, good_st = _call(head, lt, last, ws)
    assert B.workspace_error(ws) == 0 and int((good_tok >= 0).all().item()) == 1
    ws[4:8].view(torch.int32).fill_(B.DLS_DRAFT_ERR_STALLED)     # as a stalled hand-off leaves it
    tok, st = _call(head, lt, last, ws)
    assert bool((tok == -1).all().item()), tok
    assert bool(torch.isnan(st).all().item())
    assert B.workspace_error(ws) == B.DLS_DRAFT_ERR_STALLED
    ws.zero_()
    tok2, st2 = _call(head, lt, last, ws)
    assert B.workspace_error(ws) == 0
    assert torch.equal(tok2, good_tok) and torch.equal(st2.view(torch.int32), good_st.view(torch.int32))


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_prepared_buffer_of_another_head_is_refused(i):
    wl, head, lt, last = _setup(i)
    _, other, _, _ = _setup(i, seed=991)
    ws = B.draft_workspace(head, wl.batch, wl.B)
    good_tok, good_st = _call(head, lt, last, ws)
    # other's descriptor pointing at head's prepared buffer: same size, wrong tensors
    other.c.prepared = head.prepared.data_ptr()
    other.c.prepared_bytes = head.prepared.numel()
    ws2 = B.draft_workspace(head, wl.batch, wl.B)
    tok, st = _call(other, lt, last, ws2)
    assert bool((tok == -1).all().item()) and bool(torch.isnan(st).all().item())
    assert B.workspace_error(ws2) == B.DLS_DRAFT_ERR_PREPARED
    # sticky until the workspace is zero-filled
    tok, _ = _call(head, lt, last, ws2)
    assert bool((tok == -1).all().item())
    ws2.zero_()
    tok, st = _call(head, lt, last, ws2)
    assert torch.equal(tok, good_tok) and torch.equal(st.view(torch.int32), good_st.view(torch.int32))
    assert B.workspace_error(ws2) == 0 and B.workspace_error(ws) == 0


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_foreign_buffer_on_a_stalled_workspace(i):
    """Both routes report the later cause: a foreign prepared buffer over a stalled call's word."""
    wl, head, lt, last = _setup(i)
    _, other, _, _ = _setup(i, seed=991)
    other.c.prepared = head.prepared.data_ptr()
    other.c.prepared_bytes = head.prepared.numel()
    ws = B.draft_workspace(head, wl.batch, wl.B)
    ws[4:8].view(torch.int32).fill_(B.DLS_DRAFT_ERR_STALLED)
    tok, st = _call(other, lt, last, ws)
    assert bool((tok == -1).all().item()) and bool(torch.isnan(st).all().item())
    assert B.workspace_error(ws) == B.DLS_DRAFT_ERR_PREPARED


@pytest.mark.parametrize("markov,prepared,batch,adaptive", [
    (False, True, 17, False), (True, True, 33, False), (False, True, 20, True), (False, False, 17, False),
    (True, False, 3, True), (False, True, 3, True)])
def test_calls_leave_only_tagged_words(markov, prepared, batch, adaptive):
    """Calls of several shapes and routes share a workspace, whose regions move with the shape, and the
    persistent kernel trusts any word that carries its tag.  So float32 state, keys and partials may not stay
    behind: the launches per position leave the workspace as they found it, and the uncertainty pass its region
    (the last one)."""
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=20_011, d=64, H=128, r=128, B=5, batch=batch, dtype="bf16")
    if markov:
        head = B.LocalHead.markov_from_weights(*W.make_markov_head(wl.V, wl.r, "bf16", 3, scale=0.5))
    else:
        head = B.LocalHead.from_weights(W.make_head(wl, "stress"))
    if prepared:
        head.prepare()
    lt = B.as_tensor(W.make_long_logits(wl))
    last = torch.from_numpy(W.make_last_token(wl)).cuda()
    ws = B.draft_workspace(head, wl.batch, wl.B)
    B.draft_block(head, lt, last, None, 1.0, 0.5, 0.0, workspace=ws,
                  adaptive=(B.UNC_ENTROPY, 0.1, 0.7) if adaptive else None)
    torch.cuda.synchronize()
    rows = wl.batch * wl.B
    tail = (B.lib().dls_long_uncertainty_workspace_size(rows, wl.V) + 255) // 256 * 256
    assert tail > 0
    persistent = int(ws[0:4].view(torch.int32).item()) > 0   # the call epoch
    assert persistent == (prepared and batch == 3)
    left = ws[ws.numel() - tail:] if persistent else ws
    assert int(left.count_nonzero().item()) == 0


def test_error_query_is_stream_ordered():
    """dls_draft_block_error reads the word after the work queued before it on the stream."""
    wl, head, lt, last = _setup(0)
    ws = B.draft_workspace(head, wl.batch, wl.B)
    s = torch.cuda.Stream()
    out = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    with torch.cuda.stream(s):
        ws[4:8].view(torch.int32).fill_(B.DLS_DRAFT_ERR_STALLED)
        B._check(B.lib().dls_draft_block_error(B._ptr(ws), ws.numel(), B._ptr(out), B._stream(s)))
    s.synchronize()
    assert int(out.item()) == B.DLS_DRAFT_ERR_STALLED
