"""Which route a prepared call takes, and that it drafts what the oracle drafts: the persistent kernel advances
the call epoch in the first word of the workspace, the launches per position leave it.  Sizes on either side
of every line of the rule: 16 and 32 (RNN) or 32 and 48 (Markov) sequences, tiles that fill the workgroups' AGPRs
(16 x 28 x 256 = 114,688 rows at r = 256), rows of long logits at 16-byte offsets, 8 positions, H = 512, sampling."""
import functools
import math

import numpy as np
import pytest
import torch

from oracle import dels_oracle as O
from paper_2607_07409_amd import binding as B
from paper_2607_07409_amd import workloads as W
from parity_util import check_draft

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=1)
def _problem(markov, V, H, r):
    wl = W.WORKLOADS["qwen3-8b-b16"].with_(V=V, d=64, H=max(H, 8), r=r, dtype="bf16", seed=V % 1000)
    if markov:
        em, wm = W.make_markov_head(V, r, "bf16", 61, scale=math.sqrt(3.0 / math.sqrt(r)))
        return wl, B.LocalHead.markov_from_weights(em, wm).prepare(), O.MarkovHead(np.asarray(em, np.float64), np.asarray(wm, np.float64))
    hw = W.make_head(wl, "stress")
    return wl, B.LocalHead.from_weights(hw).prepare(), O.RnnHead.from_weights(hw)


@pytest.mark.parametrize("markov,V,H,r,batch,Bk,T,prior,persistent", [
    (True, 5003, 0, 128, 17, 4, 0.0, False, True),
    (True, 5003, 0, 128, 32, 4, 0.7, True, True),
    (True, 5003, 0, 128, 33, 8, 0.0, False, False),
    (True, 114_704, 0, 256, 17, 2, 0.7, True, True),
    (True, 114_704, 0, 256, 33, 8, 0.0, False, True),
    (True, 114_704, 0, 256, 48, 8, 0.7, True, True),
    (True, 114_704, 0, 256, 48, 7, 0.0, False, False),
    (True, 114_704, 0, 256, 49, 8, 0.0, True, False),
    (True, 114_701, 0, 256, 33, 8, 0.0, False, False),
    (True, 114_688, 0, 256, 33, 8, 0.0, False, False),
    (False, 5003, 128, 128, 16, 8, 0.0, False, True),
    (False, 5003, 128, 128, 17, 8, 0.0, False, False),
    (False, 114_704, 512, 256, 17, 8, 0.0, True, True),
    (False, 114_704, 512, 256, 32, 8, 0.0, False, True),
    (False, 114_704, 512, 256, 32, 8, 0.7, False, False),
    (False, 114_704, 512, 256, 33, 8, 0.0, False, False),
    (False, 114_704, 1024, 256, 17, 8, 0.0, False, False),
])
def test_route_and_parity(markov, V, H, r, batch, Bk, T, prior, persistent):
    wl, head, oracle = _problem(markov, V, H, r)
    wl = wl.with_(batch=batch, B=Bk)
    long_h, last = W.make_long_logits(wl), W.make_last_token(wl)
    pr = W.make_zipf_log_prior(V, 3) if prior else None
    be = 0.3 if prior else 0.0
    lt = B.as_tensor(long_h)
    assert head.path(batch, Bk, lt.dtype, prior) == 1
    ws = B.draft_workspace(head, batch, Bk)
    args = (head, lt, torch.from_numpy(np.asarray(last, np.int32)).cuda(),
            None if pr is None else torch.from_numpy(np.ascontiguousarray(pr, np.float32)).cuda(), 1.0, 0.5, be)
    kw = dict(workspace=ws, temperature=T, seed=11)
    tok, st = (x.clone() for x in B.draft_block(*args, **kw))
    again = B.draft_block(*args, **kw)
    torch.cuda.synchronize()
    assert B.workspace_error(ws) == 0
    assert int(ws[:4].view(torch.int32).item()) == (2 if persistent else 0)
    assert torch.equal(tok, again[0]) and torch.equal(st.view(torch.int32), again[1].view(torch.int32))
    seqs = sorted({0, 15, 16, batch // 2, batch - 1} & set(range(batch)))
    rep = check_draft(tok.cpu().numpy(), st.cpu().numpy(), oracle, long_h, last, pr, 1.0, 0.5, be, sequences=seqs,
                      temperature=T, seed=11)
    print(rep["near_ties"], rep["errs"])
    assert all(e < 2e-4 for e in rep["errs"].values()), rep["errs"]
