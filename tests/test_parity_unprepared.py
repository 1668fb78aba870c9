"""Heads drafted with by launches per position (as they are, and prepared ones of many sequences), at the sizes
where the per-position kernels change their ways: operand tiles of 16 rows and 16 sequences, chunks of 32 (bf16) or
16 (float32) columns, five hidden units per workgroup or one per wave, the vocabulary slice of a workgroup, the
register form (r <= 256) and the LDS form above, one, two, four and more tiles of sequences, and the
single-workgroup form of small heads on either side of its rule.  Tokens and
statistics against the oracle, and statistics within 2e-4 absolute: the logits here stay below about 100,
float32 products and sums keep about 1e-6 relative."""
import math

import numpy as np
import pytest
import torch

from oracle import dels_oracle as O
from paper_2607_07409_amd import binding as B
from paper_2607_07409_amd import workloads as W
from parity_util import check_draft

pytestmark = pytest.mark.gpu

CASES = [
    # V, d, H, r, B, batch, dtype, long dtype, T, prior, literal, markov
    (1, 8, 8, 8, 2, 1, "bf16", "bf16", 0.0, False, False, False),
    (15, 8, 8, 8, 3, 17, "f32", "f32", 0.0, True, True, False),
    (1024, 64, 64, 64, 4, 1, "f32", "f32", 0.0, True, False, False),
    (2049, 72, 40, 88, 5, 3, "bf16", "f32", 0.7, True, False, False),
    (1031, 0, 0, 128, 33, 5, "bf16", "bf16", 0.0, False, True, True),
    (7000, 136, 264, 96, 4, 6, "f32", "f32", 0.0, True, False, False),
    (30011, 1000, 264, 256, 4, 1, "bf16", "bf16", 0.0, False, False, False),
    (30011, 264, 1024, 136, 3, 16, "bf16", "bf16", 1.0, True, False, False),
    (20480, 520, 304, 128, 4, 17, "bf16", "f32", 0.0, True, True, False),
    (33001, 4104, 72, 248, 3, 32, "bf16", "bf16", 0.0, False, False, False),
    (16403, 256, 512, 256, 3, 33, "bf16", "bf16", 0.7, True, False, False),
    (16400, 256, 512, 256, 4, 64, "f32", "bf16", 0.0, False, False, False),
    (9001, 64, 136, 200, 3, 65, "bf16", "bf16", 0.0, True, False, False),
    (5003, 128, 128, 512, 4, 20, "bf16", "bf16", 1.0, True, False, False),
    (4099, 128, 128, 264, 3, 7, "f32", "f32", 0.0, True, True, False),
    (20011, 0, 0, 256, 4, 24, "bf16", "bf16", 0.0, True, False, True),
    (9973, 0, 0, 120, 5, 9, "f32", "f32", 0.7, False, True, True),
    (8200, 0, 0, 264, 4, 50, "bf16", "bf16", 0.0, True, False, True),
    (520_001, 8, 8, 8, 2, 3, "bf16", "bf16", 0.0, True, False, False),   # the prior's slice exceeds its LDS
    (20_011, 4104, 264, 72, 3, 2, "bf16", "bf16", 0.0, False, False, False),   # one wave per row: rounds of 2,048
    (20_011, 1064, 1032, 264, 3, 4, "f32", "f32", 0.7, True, False, False),    # (bf16) or 1,024 columns, a ragged last one
    (20_011, 2048, 520, 40, 4, 1, "f32", "bf16", 0.0, True, True, False),
    (20_011, 16, 2056, 136, 3, 3, "bf16", "bf16", 0.0, False, False, False),
    (256, 0, 0, 64, 5, 3, "bf16", "bf16", 0.0, True, False, True),             # one workgroup per sequence or launches:
    (1500, 0, 0, 64, 3, 40, "f32", "bf16", 0.7, False, True, True),            # on either side of that rule
    (1500, 0, 0, 64, 3, 3, "f32", "bf16", 0.7, False, True, True),
    (4500, 64, 64, 64, 3, 40, "bf16", "bf16", 0.0, True, True, False),
    (4500, 64, 64, 64, 3, 2, "bf16", "bf16", 0.0, True, True, False),
    (40_000, 8, 8, 8, 3, 1, "bf16", "f32", 0.7, False, False, False),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_unprepared_edges(case):
    V, d, H, r, Bk, batch, dt, ldt, T, with_prior, literal, markov = CASES[case]
    print(CASES[case], flush=True)
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=V, d=max(d, 8), H=max(H, 8), r=r, B=Bk, batch=batch, dtype=dt, seed=900 + case)
    if markov:
        em, wm = W.make_markov_head(V, r, dt, 900 + case, scale=math.sqrt(3.0 / math.sqrt(r)))
        head = B.LocalHead.markov_from_weights(em, wm)
        oracle = O.MarkovHead(np.asarray(em, np.float64), np.asarray(wm, np.float64))
    else:
        hw = W.make_head(wl, "stress")
        head, oracle = B.LocalHead.from_weights(hw), O.RnnHead.from_weights(hw)
    long_h = W.make_long_logits(wl.with_(dtype=ldt))
    last = W.make_last_token(wl)
    prior = W.make_zipf_log_prior(V, 900 + case) if with_prior else None
    al = [0.5 + 0.05 * j for j in range(Bk)]
    be = [0.3 + 0.02 * j for j in range(Bk)] if with_prior else 0.0
    lt = B.as_tensor(long_h)
    assert head.path(batch, Bk, lt.dtype, with_prior) == 0
    ws = B.draft_workspace(head, batch, Bk)
    args = (head, lt, torch.from_numpy(np.asarray(last, np.int32)).cuda(),
            None if prior is None else torch.from_numpy(np.ascontiguousarray(prior, np.float32)).cuda(), 1.0, al, be)
    kw = dict(first_row_long_only=literal, workspace=ws, temperature=T, seed=77)
    tok, st = B.draft_block(*args, **kw)
    tok, st = tok.clone(), st.clone()
    again = B.draft_block(*args, **kw)
    torch.cuda.synchronize()
    assert torch.equal(tok, again[0]) and torch.equal(st.view(torch.int32), again[1].view(torch.int32))
    rep = check_draft(tok.cpu().numpy(), st.cpu().numpy(), oracle, long_h, last, prior, 1.0, al, be, literal,
                      temperature=T, seed=77)
    print(rep["near_ties"], rep["errs"])
    assert all(e < 2e-4 for e in rep["errs"].values()), rep["errs"]


@pytest.mark.parametrize("V,r,batch", [(1024, 64, 2), (20011, 128, 20), (9001, 264, 5)])
def test_unprepared_masks_and_ties(V, r, batch):
    """-inf and lowest-value masks, a row without a finite entry, exact ties (lowest index, on positions that
    run through the vocabulary forwards and backwards) and a NaN logit, which may not hide from its row."""
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=V, d=64, H=64, r=r, B=4, batch=batch, dtype="bf16", seed=7)
    hw = W.make_head(wl, "stress")
    head, oracle = B.LocalHead.from_weights(hw), O.RnnHead.from_weights(hw)
    long_h = np.asarray(W.make_long_logits(wl), np.float32).copy()
    long_h[0, 0, ::2] = -np.inf
    long_h[0, 1, 1::3] = np.float32(-3.0e38)
    long_h[1, 2, :] = -np.inf
    for j in range(4):
        long_h[1, j, [V - 1, V // 2, 5]] = 200.0 if j != 2 else -np.inf
    last = W.make_last_token(wl)
    lt = torch.from_numpy(long_h).cuda()
    run = lambda al: B.draft_block(head, lt, torch.from_numpy(np.asarray(last, np.int32)).cuda(), None, 1.0, al, 0.0)
    tok, st = run(0.5)
    # sequence 1 holds the row without a finite entry, whose statistics are infinite
    rep = check_draft(tok.cpu().numpy(), st.cpu().numpy(), oracle, long_h, last, None, 1.0, 0.5, 0.0,
                      sequences=[b for b in range(batch) if b != 1])
    print(rep["near_ties"], rep["errs"])
    tok0, _ = run(0.0)   # no short term: the ties are exact
    assert tok0[1].tolist() == [5, 5, 0, 5]
    long_h[0, 2, V // 3] = np.nan
    lt.copy_(torch.from_numpy(long_h))
    _, st = run(0.5)
    assert torch.isnan(st[0, 2, 3]) and torch.isnan(st[0, 2, 5]) and torch.isfinite(st[0, :2, 3]).all()


@pytest.mark.parametrize("V,r,batch,T,markov,literal", [
    (5003, 128, 33, 0.0, False, True), (4099, 256, 65, 0.7, False, False), (5003, 128, 130, 0.0, False, False),
    (7001, 256, 40, 0.7, True, True), (4100, 128, 64, 0.0, True, False), (5003, 128, 17, 0.7, False, True),
    (7001, 256, 32, 0.0, False, False), (4099, 256, 17, 0.0, False, True), (5003, 128, 31, 0.7, False, False)])
def test_prepared_heads_of_many_sequences(V, r, batch, T, markov, literal):
    """Above 16 sequences (a Markov head: 32) a prepared head is drafted by launches per position: against the oracle, with the
    prior and per-position weights, the second call on the workspace bit for bit like the first."""
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=V, d=64, H=256, r=r, B=3, batch=batch, dtype="bf16", seed=40 + batch)
    if markov:
        em, wm = W.make_markov_head(V, r, "bf16", 40 + batch, scale=math.sqrt(3.0 / math.sqrt(r)))
        head = B.LocalHead.markov_from_weights(em, wm)
        oracle = O.MarkovHead(np.asarray(em, np.float64), np.asarray(wm, np.float64))
    else:
        hw = W.make_head(wl, "stress")
        head, oracle = B.LocalHead.from_weights(hw), O.RnnHead.from_weights(hw)
    head.prepare()
    long_h, last, prior = W.make_long_logits(wl), W.make_last_token(wl), W.make_zipf_log_prior(V, 3)
    al, be = [0.5, 0.55, 0.6], [0.3, 0.32, 0.34]
    lt = B.as_tensor(long_h)
    assert head.path(batch, 3, lt.dtype, True) == 1
    ws = B.draft_workspace(head, batch, 3)
    args = (head, lt, torch.from_numpy(np.asarray(last, np.int32)).cuda(),
            torch.from_numpy(np.ascontiguousarray(prior, np.float32)).cuda(), 1.0, al, be)
    kw = dict(first_row_long_only=literal, workspace=ws, temperature=T, seed=5)
    tok, st = (x.clone() for x in B.draft_block(*args, **kw))
    again = B.draft_block(*args, **kw)
    torch.cuda.synchronize()
    assert B.workspace_error(ws) == 0
    assert torch.equal(tok, again[0]) and torch.equal(st.view(torch.int32), again[1].view(torch.int32))
    alone, none = B.draft_block(*args, want_stats=False, **kw)   # tokens alone: the kernel without log-sum-exps
    assert none is None and torch.equal(alone, tok) and B.workspace_error(ws) == 0
    rep = check_draft(tok.cpu().numpy(), st.cpu().numpy(), oracle, long_h, last, prior, 1.0, al, be, literal,
                      temperature=T, seed=5)
    assert all(e < 2e-4 for e in rep["errs"].values()), rep["errs"]


@pytest.mark.parametrize("prepared,batch", [(False, 40), (True, 17), (True, 40)])
def test_log_sum_exp_precision(prepared, batch):
    """Rows of log-probabilities with one confident token: their log-sum-exp is 0, and what a kernel loses shows
    whole.  The token's own term is exactly 1 where the reference is the maximum; about thirty additions to a
    sum between 1 and 2 round by 2^-23 / sqrt(12) each, 1.9e-7 together (root mean square); a reference that lies
    30 below rounds the exponent itself by up to 2^-19."""
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=20_011, d=64, H=128, r=128, B=16, batch=batch, dtype="bf16", seed=3)
    head = B.LocalHead.from_weights(W.make_head(wl, "stress"))
    if prepared:
        head.prepare()
    g = torch.Generator().manual_seed(batch)
    x = 3.0 * torch.randn(batch * wl.B, wl.V, generator=g, dtype=torch.float64)
    x.scatter_add_(1, torch.randint(0, wl.V, (batch * wl.B, 1), generator=g), torch.full((batch * wl.B, 1), 24.0, dtype=torch.float64))
    long = torch.log_softmax(x, -1).float()
    want = long.double().logsumexp(-1)
    _, st = B.draft_block(head, long.cuda().view(batch, wl.B, wl.V), torch.from_numpy(W.make_last_token(wl)).cuda(), None,
                          1.0, 0.5, 0.0)
    err = (st.cpu().view(-1, 6)[:, B.STATS_FIELDS.index("lse_long")].double() - want).abs()
    print(prepared, batch, err.mean().item(), err.max().item())
    assert err.mean() < 3e-7


@pytest.mark.parametrize("batch,dt", [(1, "bf16"), (2, "f32"), (4, "bf16")])
def test_infinite_gate_weight(batch, dt):
    """An infinite weight in the last column closes or opens its gate; nothing past the ragged end of a row may meet it."""
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=5003, d=72, H=72, r=64, B=3, batch=batch, dtype=dt, seed=9)
    hw = W.make_head(wl, "stress")
    bits, inf = (hw.w_ih.bits, 0x7F80) if dt == "bf16" else (hw.w_ih, np.inf)
    bits[72 + 5, -1] = inf
    head, oracle = B.LocalHead.from_weights(hw), O.RnnHead.from_weights(hw)
    long_h, last = W.make_long_logits(wl), W.make_last_token(wl)
    tok, st = B.draft_block(head, B.as_tensor(long_h), torch.from_numpy(np.asarray(last, np.int32)).cuda(), None, 1.0, 0.5, 0.0)
    with np.errstate(over="ignore"):
        rep = check_draft(tok.cpu().numpy(), st.cpu().numpy(), oracle, long_h, last, None, 1.0, 0.5, 0.0)
    assert all(np.isfinite(e) and e < 2e-4 for e in rep["errs"].values()), rep["errs"]


@pytest.mark.parametrize("prepared,batch,T", [(False, 3, 0.7), (True, 20, 0.0), (True, 40, 0.7), (False, 20, 0.0)])
def test_no_long_term(prepared, batch, T):
    """w_long = 0 with masked long logits: the long term is absent, masks included, and the head and the prior
    decide alone, at one, two and four tiles of sequences."""
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=20_011, d=64, H=256, r=128, B=3, batch=batch, dtype="bf16", seed=8)
    hw = W.make_head(wl, "stress")
    head, oracle = B.LocalHead.from_weights(hw), O.RnnHead.from_weights(hw)
    if prepared:
        head.prepare()
    long_h = np.asarray(W.make_long_logits(wl), np.float32).copy()
    long_h[:, :, ::3] = -np.inf
    last, prior = W.make_last_token(wl), W.make_zipf_log_prior(wl.V, 3)
    tok, st = B.draft_block(head, torch.from_numpy(long_h).cuda(), torch.from_numpy(np.asarray(last, np.int32)).cuda(),
                            torch.from_numpy(np.ascontiguousarray(prior, np.float32)).cuda(), 0.0, 0.5, 0.3,
                            temperature=T, seed=5)
    rep = check_draft(tok.cpu().numpy(), st.cpu().numpy(), oracle, long_h, last, prior, 0.0, 0.5, 0.3, temperature=T, seed=5)
    assert all(e < 2e-4 for e in rep["errs"].values()), rep["errs"]
