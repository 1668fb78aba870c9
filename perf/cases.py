"""Workloads that a serving or training program has this library do, for timing and comparison.

A case is a dict of plain values; prepare() makes its inputs on the GPU from a seed, run() makes one
pass through the public binding, work() states the bytes and operations the pass cannot do without,
exact() computes the same outputs in float64 with plain torch.  Three kinds of work:

draft    one draft block per sequence and the acceptance lengths against the target's tokens: what a
         speculative-decoding server does between two target forwards
combine  fusion and decoding of rows whose short logits exist already (another local head, an
         evaluation of fusion weights over stored logits)
prior    the unigram log-prior of a token stream

The vocabularies, embedding widths, head sizes, block lengths and batches are those of the drafting
workloads, the tests and the benchmark of this repository; the odd ones stand for other models.
"""
import math

import torch

from paper_2607_07409_amd import binding as B
from paper_2607_07409_amd.workloads import QWEN3_VOCAB

DRAFT = dict(kind="draft", head="rnn", dtype="bf16", prepared=True, batch=1, B=16, V=QWEN3_VOCAB, d=4096, H=1024, r=256,
             alpha=0.5, beta=0.0, schedule=False, temperature=0.0, adaptive=False, exclusive=True)
COMBINE = dict(kind="combine", dtype="bf16", rows=16, V=QWEN3_VOCAB, beta=0.0, stats=True, scores=False)


def listed():
    return [
        # one user's stream, the latency case of speculative decoding (Qwen3-4B widths); the drafter has the GPU
        # to itself between target forwards
        dict(DRAFT, name="draft-b1", d=2560),
        # a few streams, the shorter block, the paper's default alpha = beta = 0.3 with the prior, per-position
        # weights, and a GPU that other work may share
        dict(DRAFT, name="draft-b3-block7-prior", batch=3, B=7, alpha=0.3, beta=0.3, schedule=True, exclusive=False),
        # serving, small batch
        dict(DRAFT, name="draft-b16", batch=16),
        # serving, the largest single-launch batch of the benchmark (Qwen3-32B width)
        dict(DRAFT, name="draft-b64", batch=64, d=5120),
        # serving at temperature 1 with the prior, a batch that fills no 16-sequence tile
        dict(DRAFT, name="draft-b40-sampled-prior", batch=40, alpha=0.3, beta=0.3, temperature=1.0, exclusive=False),
        # the Markov head with weights adapted to the entropy of the long logits
        dict(DRAFT, name="markov-b24-adaptive", head="markov", batch=24, adaptive=True, d=0, H=0),
        # a head that is drafted with as it is, without the folded 1.9 GB table: a checkpoint under evaluation, or a
        # server that has no memory left for the table
        dict(DRAFT, name="unprepared-b32", batch=32, prepared=False),
        # a float32 head of another size with float32 logits (a research model), the prior on
        dict(DRAFT, name="unprepared-f32-b6", batch=6, B=8, V=50003, d=1024, H=512, r=96, dtype="f32", prepared=False,
             alpha=0.3, beta=0.3),
        # the smallest call: the tiny float32 workload, four positions of a 1,024-word vocabulary
        dict(DRAFT, name="tiny-f32", B=4, V=1024, d=64, H=64, r=64, dtype="f32", prepared=False),
        # all rows of a batch-16 block with statistics
        dict(COMBINE, name="combine-256-stats", rows=256),
        # full score rows in float32 with the prior, an odd vocabulary (every row starts at another alignment)
        dict(COMBINE, name="combine-f32-scores", rows=48, V=32003, dtype="f32", beta=0.3, scores=True),
        # the prior of a corpus shard, estimated once per dataset
        dict(kind="prior", name="prior-20M", n=20_000_003, V=QWEN3_VOCAB),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5))))))


def draw(rng):
    """One more case of the same ranges."""
    pick = rng.random()
    if pick < 0.42:      # prepared heads: batches 1 to 64, both ranks, every decoding option
        c = dict(DRAFT, batch=_log(rng, 1, 64), B=rng.choice([4, 5, 7, 8, 11, 16, 16]), d=rng.choice([2560, 4096, 5120]),
                 V=rng.choice([QWEN3_VOCAB, QWEN3_VOCAB, _log(rng, 30011, 151000)]), r=rng.choice([256, 256, 128]),
                 exclusive=rng.random() < 0.6)
        if rng.random() < 0.25:
            c.update(head="markov", d=0, H=0)
    elif pick < 0.68:    # heads as they are: any width that is a multiple of 8, both types
        c = dict(DRAFT, prepared=False, batch=_log(rng, 1, 32), B=rng.choice([4, 7, 8, 16]),
                 dtype=rng.choice(["bf16", "bf16", "f32"]), V=_log(rng, 1024, 152000), d=8 * _log(rng, 8, 512),
                 H=8 * _log(rng, 8, 128), r=8 * _log(rng, 4, 32), exclusive=rng.random() < 0.5)
        if c["dtype"] == "f32":
            c.update(batch=min(c["batch"], 12), V=min(c["V"], 64000))
        if rng.random() < 0.2:
            c.update(head="markov", d=0, H=0)
    elif pick < 0.9:
        c = dict(COMBINE, dtype=rng.choice(["bf16", "bf16", "f32"]), rows=_log(rng, 4, 1024), V=_log(rng, 5003, 152000),
                 beta=rng.choice([0.0, 0.3]), stats=rng.random() < 0.7)
        c["scores"] = c["stats"] and rng.random() < 0.3
        c["rows"] = max(4, min(c["rows"], 60_000_000 // c["V"]))
    else:
        c = dict(kind="prior", n=_log(rng, 100_003, 20_000_000), V=_log(rng, 5003, 152000))
    if c["kind"] == "draft":
        if rng.random() < 0.4:
            c.update(alpha=0.3, beta=0.3)
        c["schedule"] = rng.random() < 0.25
        c["temperature"] = rng.choice([0.0, 0.0, 0.7, 1.0])
        c["adaptive"] = rng.random() < 0.2
    return c


# ----------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _normal(shape, std, dtype, g):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _logits(rows, V, dtype, g):
    """Rows of model logits: 3 N(0, 1) with one token raised, by 16 where the model is sure (three rows in
    four), by 8 elsewhere, where the local head and the noise of the other 150,000 decide."""
    x = _normal((rows, V), 3.0, dtype, g)
    top = torch.randint(0, V, (rows, 1), device="cuda", generator=g)
    lift = torch.where(torch.rand((rows, 1), device="cuda", generator=g) < 0.75, 16.0, 8.0)
    return x.scatter_(1, top, (x.gather(1, top).float() + lift).to(dtype))


def _zipf_prior(V, g):
    ranks = torch.randperm(V, device="cuda", generator=g).double() + 1.0
    return torch.log_softmax(-1.1 * ranks.log(), 0).float()


def _weights(case, g):
    """Head weights at the scale of a trained head: short logits with a spread of a few units."""
    V, d, H, r, dt = case["V"], case["d"], case["H"], case["r"], _dt(case)
    if case["head"] == "markov":
        s = math.sqrt(3.0 / math.sqrt(r))
        return _normal((V, r), s, dt, g), _normal((V, r), s, dt, g)
    return (_normal((V, d), 1.0, dt, g), _normal((3 * H, d), 1.0 / math.sqrt(d), dt, g),
            _normal((3 * H, H), 1.0 / math.sqrt(H), dt, g), _normal((r, H), 1.0 / math.sqrt(H), dt, g),
            _normal((V, r), 10.0 / math.sqrt(r), dt, g))


def _fusion(case):
    """alpha and beta: scalars, or rising with the position like the learned per-position weights."""
    if not case["schedule"]:
        return case["alpha"], case["beta"]
    al = [case["alpha"] + 0.02 * j for j in range(case["B"])]
    return al, ([case["beta"] + 0.01 * j for j in range(case["B"])] if case["beta"] else 0.0)


RULE = (B.UNC_ENTROPY, 0.1, 0.7)


def prepare(case, seed):
    g = _gen(seed)
    V = case["V"]
    if case["kind"] == "prior":
        order = torch.randperm(V, device="cuda", generator=g).int()
        cdf = torch.cumsum(torch.arange(1, V + 1, device="cuda", dtype=torch.float64) ** -1.1, 0)
        u = torch.rand(case["n"], device="cuda", generator=g, dtype=torch.float64) * cdf[-1]
        return dict(case=case, tokens=order[torch.searchsorted(cdf, u).clamp_(max=V - 1)])
    if case["kind"] == "combine":
        rows, dt = case["rows"], _dt(case)
        long = _logits(rows, V, dt, g)
        short = _normal((rows, V), 3.0, dt, g)
        out = (torch.empty(rows, dtype=torch.int32, device="cuda"),
               torch.empty((rows, 6), device="cuda") if case["stats"] else None,
               torch.empty((rows, V), device="cuda") if case["scores"] else None)
        ws = torch.empty(max(256, B.combine_logits_workspace_size(rows, V)), dtype=torch.uint8, device="cuda")
        return dict(case=case, long=long, short=short, out=out, ws=ws,
                    prior=_zipf_prior(V, g) if case["beta"] else None)
    batch, Bk = case["batch"], case["B"]
    w = _weights(case, g)
    head = B.LocalHead.markov(*w) if case["head"] == "markov" else B.LocalHead(*w)
    if case["prepared"]:
        head.prepare()
    long = _logits(batch * Bk, V, _dt(case), g).view(batch, Bk, V)
    last = torch.randint(0, V, (batch,), device="cuda", generator=g, dtype=torch.int32)
    # the target model agrees with the long logits' own choice on part of the positions
    target = long.argmax(-1).int()
    other = torch.randint(0, V, (batch, Bk), device="cuda", generator=g, dtype=torch.int32)
    target = torch.where(torch.rand((batch, Bk), device="cuda", generator=g) < 0.8, target, other).contiguous()
    return dict(case=case, head=head, long=long, last=last, target=target, seed=seed * 0x9E3779B97F4A7C15 % (1 << 64),
                prior=_zipf_prior(V, g) if case["beta"] else None, ws=B.draft_workspace(head, batch, Bk),
                out=(torch.empty((batch, Bk), dtype=torch.int32, device="cuda"),
                     torch.empty((batch, Bk, 6), device="cuda")),
                unc=torch.empty((batch, Bk, 4), device="cuda") if case["adaptive"] else None,
                acc=torch.empty(batch, dtype=torch.int32, device="cuda"))


def run(state):
    case = state["case"]
    if case["kind"] == "prior":
        logp, counts = B.unigram_log_prior(state["tokens"], case["V"])
        return dict(log_prior=logp, counts=counts)
    if case["kind"] == "combine":
        tok, st, sc = B.combine_logits(state["long"], state["short"], state["prior"], 1.0, 0.3, case["beta"],
                                       out=state["out"], workspace=state["ws"])
        return dict(tokens=tok, stats=st, scores=sc)
    al, be = _fusion(case)
    got = B.draft_block(state["head"], state["long"], state["last"], state["prior"], 1.0, al, be, out=state["out"],
                        workspace=state["ws"], temperature=case["temperature"], seed=state["seed"],
                        exclusive_device=case["exclusive"], adaptive=RULE if case["adaptive"] else None,
                        out_uncertainty=state["unc"])
    acc = B.accept_len(got[0], state["target"], out=state["acc"])
    return dict(tokens=got[0], stats=got[1], uncertainty=got[2] if case["adaptive"] else None, accepted=acc)


# ----------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------
def work(case):
    V = case["V"]
    if case["kind"] == "prior":
        return dict(bytes=4 * case["n"] + 12 * V, flops=case["n"])
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "combine":
        rows = case["rows"]
        return dict(bytes=rows * V * (2 * e + (4 if case["scores"] else 0)) + (4 * V if case["beta"] else 0) +
                    rows * (4 + 24 * case["stats"]), flops=rows * V * (4 + 12 * case["stats"]))
    n, H, r, d = case["batch"] * case["B"], case["H"], case["r"], case["d"]
    weights, per = V * r, V * r                      # elements read once; products per drafted token
    if case["head"] == "rnn":
        weights += 3 * H * H + r * H + (0 if case["prepared"] else 3 * H * d)
        per += 3 * H * H + r * H + (0 if case["prepared"] else 3 * H * d)
    # a row of the folded table, of E or of E_M for each drafted token
    row = (4 * 3 * H if case["prepared"] else e * d) if case["head"] == "rnn" else e * r
    return dict(bytes=weights * e + n * (row + V * e + 28) + (4 * V if case["beta"] else 0), flops=2 * per * n + 16 * n * V)


def tolerance(case):
    if case["kind"] == "prior":
        return dict(rel=1e-7)    # float64 logarithms rounded once
    # float32 sums of exponentials and products: up to 5e-7 from float64 over these ranges on either path, and
    # two orders of summation are two such errors apart; a drafted token may fall to the other side of a tie
    return dict(rel=4e-6, max=4e-5, differ=0.005)


# ----------------------------------------------------------------------------------------------
# the same in float64
# ----------------------------------------------------------------------------------------------
def _mul32(m, c):
    """High and low words of a 32 x 32-bit product (int64 tensors; the product wraps, its bits do not)."""
    p = c * m
    return (p >> 32) & 0xFFFFFFFF, p & 0xFFFFFFFF


def _gumbel(seed, j, batch, V):
    """[batch, V] standard Gumbel noise: word v % 4 of Philox4x32-10 at counter (v / 4, j, b, 0)."""
    q = torch.arange((V + 3) // 4, device="cuda", dtype=torch.int64).expand(batch, -1)
    b = torch.arange(batch, device="cuda", dtype=torch.int64)[:, None].expand_as(q)
    c = [q, torch.full_like(q, j), b, torch.zeros_like(q)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        h0, l0 = _mul32(0xD2511F53, c[0])
        h1, l1 = _mul32(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    x = torch.stack(c, -1).view(batch, -1)[:, :V]
    u = ((x >> 9).double() + 0.5) * 2.0 ** -23
    return -torch.log(-torch.log(u))


def _stats(long, short, fused, norm, temperature=0.0, noise=None):
    scaled = fused / temperature if temperature else fused
    decide = scaled + noise if noise is not None else scaled
    tok = decide.float().argmax(-1)
    top = decide.topk(2, -1).values
    lse_f = scaled.logsumexp(-1)
    at = tok[:, None]
    return tok, torch.stack([fused.gather(1, at)[:, 0] - norm, scaled.gather(1, at)[:, 0] - lse_f, top[:, 0] - top[:, 1],
                             long.logsumexp(-1), short.logsumexp(-1), lse_f], -1)


def exact(case, seed):
    s = prepare(case, seed)
    V = case["V"]
    prior = s["prior"].double() if s.get("prior") is not None else torch.zeros(V, dtype=torch.float64, device="cuda")
    if case["kind"] == "prior":
        counts = torch.bincount(s["tokens"].long(), minlength=V)
        logp = torch.log((counts.double() + 1.0) / (case["n"] + float(V)))
        return dict(log_prior=logp, counts=torch.cat([counts, counts.sum()[None]]))
    if case["kind"] == "combine":
        toks, sts, scs = [], [], []
        for a, b in zip(s["long"].split(64), s["short"].split(64)):
            a, b = a.double(), b.double()
            f = a + _f32(0.3) * b - _f32(case["beta"]) * prior
            norm = a.logsumexp(-1) + _f32(0.3) * b.logsumexp(-1)
            tok, st = _stats(a, b, f, norm)
            toks.append(tok.int())
            sts.append(st)
            if case["scores"]:
                scs.append(f - norm[:, None])
        return dict(tokens=torch.cat(toks), stats=torch.cat(sts) if case["stats"] else None,
                    scores=torch.cat(scs) if case["scores"] else None)
    batch, Bk, H, head = case["batch"], case["B"], case["H"], s["head"]
    al, be = _fusion(case)
    w_v = head.w_vocab.double()
    if case["head"] == "rnn":
        w_ih, w_hh, w_rank = head.w_ih.double(), head.w_hh.double(), head.w_rank.double()
        h = torch.zeros((batch, H), dtype=torch.float64, device="cuda")
    u, toks, sts, uncs = s["last"].long(), [], [], []
    for j in range(Bk):
        x = head.emb[u].double()
        if case["head"] == "rnn":
            gi, gh = x @ w_ih.T, h @ w_hh.T
            rg = torch.sigmoid(gi[:, :H] + gh[:, :H])
            zg = torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
            ng = torch.tanh(gi[:, 2 * H:] + rg * gh[:, 2 * H:])
            h = (1.0 - zg) * ng + zg * h
            x = h @ w_rank.T
            x = x * torch.sigmoid(x)
        short = x @ w_v.T
        long = s["long"][:, j].double()
        a = torch.full((batch, 1), _f32(al[j] if case["schedule"] else al), dtype=torch.float64, device="cuda")
        b = torch.full((batch, 1), _f32(be[j] if case["schedule"] and case["beta"] else be), dtype=torch.float64, device="cuda")
        if case["adaptive"]:
            lp = torch.log_softmax(long, -1)
            ent = -(lp.exp() * lp).sum(-1)
            uu = ent / math.log(V)
            gate = ((uu - _f32(RULE[1])) / (_f32(RULE[2]) - _f32(RULE[1]))).clamp(0.0, 1.0)
            uncs.append(torch.stack([ent, lp.max(-1).values.exp(), uu, gate], -1))
            a, b = a * gate[:, None], b * gate[:, None]
        f = long + a * short - b * prior
        norm = long.logsumexp(-1) + a[:, 0] * short.logsumexp(-1)
        T = case["temperature"]
        u, st = _stats(long, short, f, norm, _f32(T), _gumbel(s["seed"], j, batch, V) if T else None)
        toks.append(u.int())
        sts.append(st)
    tok = torch.stack(toks, 1)
    acc = (tok == s["target"]).int().cumprod(1).sum(1).int()
    return dict(tokens=tok, stats=torch.stack(sts, 1), uncertainty=torch.stack(uncs, 1) if case["adaptive"] else None,
                accepted=acc)


def _f32(x):
    """A weight as the library receives it."""
    return float(torch.tensor(x, dtype=torch.float32))
