"""Performance cases: the calls a program using this framework makes, over the sizes it
makes them at.

A case is a dict of plain values.  Its `kind` names the entry point:

  chain      one verify-and-arbitrate step over chain blocks (`prepare_block(...).launch()`)
  rollout    the chain step in two phases around the caller's arbitrator, at temperature 1
             with sampled arbitration and the reinforcement-learning statistics
             (`SplitBlock`, then its `arbitrate`)
  tree       one verify step over token trees (`prepare_tree(...).launch()`)
  sps        the speculative-sampling baseline (`prepare_sps(...).launch()`)
  attention  the arbitrator's hybrid attention (`hybrid_attention`), for one round's region
             queries (`form` "round") or for a whole input (`form` "prefill")
  arbitrate  the arbitration head alone on selected hidden rows (`arbitrate`)

Logits are N(0, 1) * 4 with a peak on some rows, and the draft's are the target's plus
noise, as in the named workloads of `paper_2605_24793_amd.workloads`; rows that are sampled
at temperature 1 all carry a peak of varying height, since a language model's
distributions are mostly far from flat there.  Everything is made on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

import paper_2605_24793_amd as cs
from paper_2605_24793_amd.workloads import Head

_BF16, _F32 = "bf16", "f32"


def listed():
    return [
        # one interactive user: latency is everything
        dict(name="chain_tiny_f32", kind="chain", B=1, K=4, V=32000, dtype=_F32, d=512, h=128, bias=False,
             packed=False, lam=0.5),
        # a handful of users with a LLaMA-3 sized vocabulary
        dict(name="chain_small", kind="chain", B=8, K=5, V=128256, dtype=_BF16, d=4096, h=256, bias=False,
             packed=False, lam=0.5),
        # a serving batch with a Qwen3 sized vocabulary
        dict(name="chain_serving", kind="chain", B=64, K=7, V=151936, dtype=_BF16, d=4096, h=256, bias=False,
             packed=False, lam=0.5),
        # the largest serving batch, the shape the framework's headline rate is quoted on
        dict(name="chain_large", kind="chain", B=256, K=7, V=151936, dtype=_BF16, d=5120, h=512, bias=False,
             packed=False, lam=0.5),
        # longer blocks over an odd vocabulary in padded rows, hidden states packed as the
        # arbitrator leaves them, a head with biases
        dict(name="chain_ragged_packed", kind="chain", B=16, K=15, V=50001, dtype=_BF16, d=4096, h=256, bias=True,
             packed=True, lam=0.3),
        # reinforcement-learning rollouts at the paper's block length
        dict(name="rollout_split", kind="rollout", B=48, K=25, V=128256, dtype=_BF16, d=4096, h=256, bias=False,
             packed=True, lam=0.5),
        # token trees: 4 children of the root, then 11 nodes a level, 60 nodes
        dict(name="tree", kind="tree", B=64, depth=6, V=151936, dtype=_BF16, d=4096, h=256, bias=False, lam=0.5),
        # the speculative-sampling baseline
        dict(name="sps", kind="sps", B=128, K=7, V=151936, dtype=_BF16),
        # the arbitrator's attention in one round of a serving batch (context lengths vary)
        dict(name="attention_round", kind="attention", form="round", B=64, ctx=2048, K=7, Hq=32, Hkv=8, D=128),
        # the same for two users with long contexts
        dict(name="attention_long", kind="attention", form="round", B=2, ctx=16384, K=7, Hq=32, Hkv=8, D=128),
        # the arbitrator's first pass over whole inputs
        dict(name="attention_prefill", kind="attention", form="prefill", B=4, ctx=2048, K=7, Hq=32, Hkv=8, D=128),
        # the head alone over the scored positions of many rounds, as training evaluates it
        dict(name="arbitrate_rows", kind="arbitrate", rows=6000, n_sel=4096, dtype=_BF16, d=5120, h=512, bias=True,
             lam=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(512, 128), (1024, 128), (2048, 256), (2560, 320), (4096, 256), (5120, 512)]


def draw(rng):
    kind = rng.choice(["chain", "chain", "chain", "rollout", "tree", "sps", "attention", "attention", "attention",
                       "arbitrate"])
    dtype = rng.choice([_BF16, _BF16, _BF16, _F32])
    d, h = rng.choice(_HEADS)
    bias = rng.random() < 0.5
    lam = rng.choice([0.3, 0.5, 0.7])
    vocab = rng.choice([32000, 32001, 50001, 128256, 151936, _log_int(rng, 4000, 152000)])
    most = 1.1e9                                       # logit bytes of a drawn step
    eb = 2 if dtype == _BF16 else 4
    if kind in ("chain", "rollout", "sps"):
        K = rng.choice([1, 3, 4, 5, 7, 10, 15, 20, 25, rng.randint(1, 40)])
        B = max(1, min(_log_int(rng, 1, 256), int(most / ((2 * K + 1) * vocab * eb))))
        if kind == "sps":
            return dict(kind=kind, B=B, K=K, V=vocab, dtype=dtype)
        return dict(kind=kind, B=B, K=K, V=vocab, dtype=dtype, d=d, h=h, bias=bias, packed=rng.random() < 0.4, lam=lam)
    if kind == "tree":
        depth = rng.randint(2, 8)
        n = 1 + 4 + 11 * (depth - 1)
        B = max(1, min(_log_int(rng, 1, 64), int(most / (2 * n * vocab * eb))))
        return dict(kind=kind, B=B, depth=depth, V=vocab, dtype=dtype, d=d, h=h, bias=bias, lam=lam)
    if kind == "attention":
        Hq, Hkv = rng.choice([(32, 8), (32, 8), (16, 4), (16, 8), (28, 4), (8, 8)])
        D = rng.choice([128, 128, 64])
        K = rng.choice([4, 5, 7, 15, 25])
        if rng.random() < 0.35:
            ctx = _log_int(rng, 100, 2048)
            B = max(1, min(_log_int(rng, 1, 16), int(4 * 2048.0 ** 2 / ctx ** 2)))
            return dict(kind=kind, form="prefill", B=B, ctx=ctx, K=K, Hq=Hq, Hkv=Hkv, D=D)
        ctx = _log_int(rng, 200, 20000)
        B = max(1, min(_log_int(rng, 1, 64), 64 * 2048 // ctx))
        return dict(kind=kind, form="round", B=B, ctx=ctx, K=K, Hq=Hq, Hkv=Hkv, D=D)
    n_sel = _log_int(rng, 8, 4096)
    return dict(kind="arbitrate", rows=int(n_sel * rng.uniform(1.0, 1.5)), n_sel=n_sel, dtype=dtype, d=d, h=h,
                bias=bias, lam=lam)


# --------------------------------------------------------------------------- inputs

def _dt(name):
    return torch.bfloat16 if name == _BF16 else torch.float32


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda")


def _rows(g, B, R, V, dt):
    """[B, R, V] rows of an element type, spaced so that each starts on 16 bytes."""
    per = 16 // torch.empty(0, dtype=dt).element_size()
    ld = (V + per - 1) // per * per
    return torch.zeros(B, R, ld, dtype=dt, device="cuda")[:, :, :V]


def _logits(g, B, RT, RD, V, dt, all_peaked):
    """Target rows [B, RT, V] and draft rows [B, RD, V], draft row j about target row j."""
    target, draft = _rows(g, B, RT, V, dt), _rows(g, B, RD, V, dt)
    sigma = 0.3 + 1.7 * _rand(g, B)
    step = max(1, int(2e8 // (RT * V)))
    for b in range(0, B, step):
        n = min(step, B - b)
        t = _randn(g, n, RT, V).mul_(4.0)
        at = (_rand(g, n, RT, 1) * V).long().clamp_(max=V - 1)
        if all_peaked:
            peak = 16.0 + 10.0 * _rand(g, n, RT, 1)
        else:
            peak = 12.0 * (_rand(g, n, RT, 1) < 0.2)
        t.scatter_add_(2, at, peak)
        target[b:b + n] = t.to(dt)
        if RD:
            draft[b:b + n] = t[:, :RD].add_(_randn(g, n, RD, V).mul_(sigma[b:b + n, None, None])).to(dt)
        del t
    return target, draft


def _sampled(g, rows):
    """One token per row of [B, R, V], drawn from its softmax."""
    B, R, V = rows.shape
    out = torch.empty(B, R, dtype=torch.int32, device="cuda")
    for b in range(B):
        x = rows[b].float()
        out[b] = (x - torch.log(-torch.log(_rand(g, R, V).clamp_(1e-12, 1 - 1e-7)))).argmax(-1).int()
    return out


def _greedy(rows):
    B, R, V = rows.shape
    return torch.stack([rows[b].float().argmax(-1).int() for b in range(B)])


def _head(g, c):
    d, h, dt = c["d"], c["h"], _dt(c["dtype"])
    w1 = (_randn(g, h, d) / math.sqrt(d)).to(dt)
    w2 = (_randn(g, h) / math.sqrt(h)).to(dt)
    b1, b2 = None, 0.0
    if c["bias"]:
        b1, b2 = (_randn(g, h) * 0.5).to(dt), 0.125
    return Head(w1, b1, w2, b2)


def _chain_inputs(c, seed, all_peaked):
    g = _gen(seed)
    B, K, V, dt = c["B"], c["K"], c["V"], _dt(c["dtype"])
    s = dict(case=c)
    s["target"], s["draft"] = _logits(g, B, K + 1, K, V, dt, all_peaked)
    s["tokens"] = _sampled(g, s["draft"]) if all_peaked else _greedy(s["draft"])
    if c["kind"] != "sps":
        s["head"] = _head(g, c)
        if c["packed"]:
            # one row per position of every sequence's [SEP, draft, SEP, candidates, SEP] region
            s["hidden"] = _randn(g, B * (2 * K + 3), c["d"]).to(dt)
            s["row0"] = torch.arange(B, dtype=torch.int64, device="cuda") * (2 * K + 3) + 1
        else:
            s["hidden"] = _randn(g, B, K, c["d"]).to(dt)
            s["row0"] = None
    return g, s


def _tree_inputs(c, seed):
    """Trees grown from the draft rows: the root's 4 best tokens, then the 11 best of
    every level's children by cumulative log-probability."""
    g = _gen(seed)
    N = 1 + 4 + 11 * (c["depth"] - 1)
    B, V, dt = c["B"], c["V"], _dt(c["dtype"])
    s = dict(case=c)
    s["target"], s["draft"] = _logits(g, B, N, N, V, dt, False)
    top = torch.empty(B, N, 4, dtype=torch.int64)
    logp = torch.empty(B, N, 4)
    for b in range(B):
        x = s["draft"][b].float()
        v, i = torch.topk(x, 4, dim=-1)
        top[b], logp[b] = i.cpu(), (v - torch.logsumexp(x, -1, keepdim=True)).cpu()
    top, logp = top.tolist(), logp.tolist()
    parent, token = [], []
    for b in range(B):
        par, tok, cum, level = [-1], [-1], [0.0], [0]
        for lev in range(1, c["depth"] + 1):
            cand = [(cum[p] + logp[b][p][r], p, r) for p in level for r in range(4)]
            if lev > 1:
                cand = sorted(cand, key=lambda t: (-t[0], t[1], t[2]))[:11]
            level = []
            for score, p, r in sorted(cand, key=lambda t: (t[1], t[2])):
                level.append(len(par))
                par.append(p)
                tok.append(top[b][p][r])
                cum.append(score)
        parent.append(par)
        token.append(tok)
    s["parent"] = torch.tensor(parent, dtype=torch.int32, device="cuda")
    s["tokens"] = torch.tensor(token, dtype=torch.int32, device="cuda")
    s["head"] = _head(g, c)
    s["hidden"] = _randn(g, B, N, c["d"]).to(dt)
    return s


def _ctx_len(c, b):
    """Context length of sequence b: from half of the longest to the longest."""
    return c["ctx"] if c["B"] == 1 else c["ctx"] - (c["ctx"] // 2) * b // (c["B"] - 1)


def _attention_inputs(c, seed):
    g = _gen(seed)
    B, K, Hq, Hkv, D = c["B"], c["K"], c["Hq"], c["Hkv"], c["D"]
    L = c["ctx"] + 2 * K + 3
    n_q = L if c["form"] == "prefill" else 2 * K + 3
    s = dict(case=c, scale=1.0 / math.sqrt(D))
    for name, n, heads in (("q", n_q, Hq), ("k", L, Hkv), ("v", L, Hkv)):
        s[name] = _randn(g, B, n, heads, D).to(torch.bfloat16)
    s["ctx_len"] = torch.tensor([_ctx_len(c, b) for b in range(B)], dtype=torch.int32, device="cuda")
    s["q_start"] = torch.zeros_like(s["ctx_len"]) if c["form"] == "prefill" else s["ctx_len"].clone()
    return s


def _arbitrate_inputs(c, seed):
    g = _gen(seed)
    s = dict(case=c)
    s["hidden"] = _randn(g, c["rows"], c["d"]).to(_dt(c["dtype"]))
    s["index"] = torch.argsort(_rand(g, c["rows"]))[:c["n_sel"]].sort().values.int()
    s["head"] = _head(g, c)
    return s


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind == "chain":
        g, s = _chain_inputs(c, seed, False)
        s["step"] = cs.prepare_block(s["target"], s["draft"], s["tokens"], s["hidden"], s["head"], c["lam"],
                                     hidden_row0=s["row0"])
    elif kind == "rollout":
        g, s = _chain_inputs(c, seed, True)
        s["sample_u"] = _rand(g, c["B"], c["K"] + 1)
        s["policy_u"] = _rand(g, c["B"], c["K"])
        s["correct"] = (_rand(g, c["B"]) < 0.5).to(torch.uint8)
    elif kind == "tree":
        s = _tree_inputs(c, seed)
        s["step"] = cs.prepare_tree(s["target"], s["draft"], s["parent"], s["tokens"], s["hidden"], s["head"], c["lam"])
    elif kind == "sps":
        g, s = _chain_inputs(c, seed, True)
        s["uniforms"] = _rand(g, c["B"], c["K"] + 1)
        s["step"] = cs.prepare_sps(s["target"], s["draft"], s["tokens"], s["uniforms"])
    elif kind == "attention":
        s = _attention_inputs(c, seed)
    else:
        s = _arbitrate_inputs(c, seed)
    return s


def run(state):
    s = state
    c = s["case"]
    kind = c["kind"]
    if kind == "attention":
        return cs.hybrid_attention(s["q"], s["k"], s["v"], s["ctx_len"], s["q_start"], c["K"], s["scale"])
    if kind == "arbitrate":
        return cs.arbitrate(s["hidden"], s["head"], c["lam"], s["index"])
    if kind == "rollout":
        # the caller's arbitrator would run between the two phases; its hidden states are given
        split = cs.SplitBlock(s["target"], s["draft"], s["tokens"], s["head"], sample_u=s["sample_u"])
        return split.arbitrate(s["hidden"], c["lam"], policy_u=s["policy_u"], correct=s["correct"],
                               hidden_row0=s["row0"])
    s["step"].launch()
    return s["step"].result()


# --------------------------------------------------------------------- what a pass needs

def _tree_nodes(c):
    return 1 + 4 + 11 * (c["depth"] - 1)


def work(case):
    c = case
    kind = c["kind"]
    if kind == "attention":
        nbytes = flops = 0
        for b in range(c["B"]):
            ctx = _ctx_len(c, b)
            n = ctx + 2 * c["K"] + 3
            region = 2 * c["K"] + 3
            rows = (c["ctx"] + region) if c["form"] == "prefill" else region
            pairs = region * n + (ctx * (ctx + 1) // 2 if c["form"] == "prefill" else 0)
            nbytes += 2 * n * c["Hkv"] * c["D"] * 2 + 2 * rows * c["Hq"] * c["D"] * 2
            flops += 4 * pairs * c["Hq"] * c["D"]
        return {"bytes": nbytes, "flops": flops}
    eb = 2 if c["dtype"] == _BF16 else 4
    if kind == "arbitrate":
        return {"bytes": c["n_sel"] * (c["d"] * eb + 9) + c["h"] * (c["d"] + 2) * eb,
                "flops": 2 * c["n_sel"] * c["d"] * c["h"]}
    if kind == "tree":
        # the draft rows of nodes with a child: the root's and about half of the others'
        rows, dec = c["B"] * (_tree_nodes(c) + 1 + _tree_nodes(c) // 2), c["B"] * (_tree_nodes(c) - 1)
    else:
        rows, dec = c["B"] * (2 * c["K"] + 1), c["B"] * c["K"]
    nbytes, flops = rows * c["V"] * eb + rows * 20 + dec * 24, 4 * rows * c["V"]
    if kind != "sps":
        scored = dec // 2                              # the mismatches are what the head must read
        nbytes += scored * c["d"] * eb + c["h"] * (c["d"] + 2) * eb
        flops += 2 * scored * c["d"] * c["h"]
    else:
        nbytes += 2 * c["B"] * c["V"] * eb             # the last token's two rows, known only after the first read
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "attention":
        # the attention weights enter the second product in bf16 and the result is bf16
        return {"rel": 1e-2, "max": 0.1}
    # 32-bit sums; temperature-1 draws may land on the neighbour of a cumulative boundary
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.005 if kind in ("rollout", "sps") else 0.001}


# --------------------------------------------------------------------- 64-bit results

def _row_stats(rows):
    """max, first argmax, log sum exp and entropy of [B, R, V] rows, in 64 bits."""
    B, R, V = rows.shape
    mx, lse, ent = (torch.empty(B, R, dtype=torch.float64, device="cuda") for _ in range(3))
    arg = torch.empty(B, R, dtype=torch.int64, device="cuda")
    idx = torch.arange(V, device="cuda")
    for b in range(B):
        for r in range(0, R, 32):
            x = rows[b, r:r + 32].double()
            m = x.amax(-1, keepdim=True)
            arg[b, r:r + 32] = torch.where(x == m, idx, V).amin(-1)
            e = torch.exp(x - m)
            S = e.sum(-1, keepdim=True)
            mx[b, r:r + 32], lse[b, r:r + 32] = m[:, 0], (m + S.log())[:, 0]
            ent[b, r:r + 32] = (S.log()[:, 0] - (e * (x - m)).sum(-1) / S[:, 0])
    return mx, arg, lse, ent


def _drawn(rows, lse, u):
    """The smallest index of each row whose cumulative probability exceeds u."""
    B, R, V = rows.shape
    out = torch.empty(B, R, dtype=torch.int64, device="cuda")
    for b in range(B):
        cum = torch.exp(rows[b].double() - lse[b][:, None]).cumsum(-1)
        out[b] = (cum <= u[b].double()[:, None] * cum[:, -1:]).sum(-1).clamp(max=V - 1)
    return out


def _scores(hidden, head):
    z = torch.empty(hidden.shape[0], dtype=torch.float64, device="cuda")
    w1, w2 = head.w1.double().t().contiguous(), head.w2.double()
    for r in range(0, hidden.shape[0], 4096):
        u = hidden[r:r + 4096].double() @ w1
        if head.b1 is not None:
            u = u + head.b1.double()
        z[r:r + 4096] = u.clamp_(min=0) @ w2 + head.b2
    return z


def _at(rows, tok):
    return torch.stack([rows[b].gather(1, tok[b].long()[:, None])[:, 0].double() for b in range(rows.shape[0])])


def _verdicts(z, match, lam, policy_u):
    """z_tilde, policy, accept and logp_action of decisions with logits z."""
    pi = torch.sigmoid(z)
    acc = match | ((policy_u.double() < pi) if policy_u is not None else (pi > lam))
    la = torch.where(acc, torch.nn.functional.logsigmoid(z), torch.nn.functional.logsigmoid(-z))
    inf = torch.full_like(z, math.inf)
    return (torch.where(match, inf, z), torch.where(match, torch.ones_like(z), pi), acc,
            torch.where(match, torch.zeros_like(z), la))


def _exact_chain(c, s):
    B, K = c["B"], c["K"]
    tmax, targ, tlse, tent = _row_stats(s["target"])
    dmax, darg, dlse, dent = _row_stats(s["draft"])
    tok = s["tokens"].long()
    lt = _at(s["target"][:, :K], tok) - tlse[:, :K]
    ld = _at(s["draft"], tok) - dlse
    out = dict(accept_len=None, tokens=None, tgt_argmax=None, tgt_max=tmax, tgt_lse=tlse, tgt_entropy=tent,
               drf_argmax=None, drf_max=dmax, drf_lse=dlse, drf_entropy=dent, logp_tgt=lt, logp_drf=ld, delta=None,
               accept=None, tgt_candidate=None)
    if c["kind"] == "sps":
        out["policy"] = torch.exp(lt - ld).clamp(max=1.0)
        return out
    cand = targ if c["kind"] == "chain" else _drawn(s["target"], tlse, s["sample_u"])
    hidden = s["hidden"]
    if s["row0"] is None:
        hidden = hidden.reshape(B * K, -1)
    else:
        hidden = hidden[(s["row0"][:, None] + torch.arange(K, device="cuda")).reshape(-1)]
    z = _scores(hidden, s["head"]).reshape(B, K)
    match = tok == cand[:, :K]
    policy_u = s.get("policy_u")
    out["z_tilde"], out["policy"], acc, out["logp_action"] = _verdicts(z, match, c["lam"], policy_u)
    if c["kind"] == "rollout":
        i = torch.arange(1, K + 1, device="cuda")
        stop = torch.where(acc, K + 1, i).amin(1)                      # s of every round
        mism = ~match
        first = torch.where(mism, i, K + 1).amin(1)
        rho = torch.where(first <= K, (stop - first).double() / (K + 1 - first).double(), math.nan)
        eff = mism & (i <= stop[:, None]) & (i <= K)
        failed = torch.where(acc, -1.0 * lt.abs(), torch.full_like(lt, -0.25))
        reward = torch.where(eff, torch.where(s["correct"].bool()[:, None], rho[:, None], failed), torch.zeros_like(lt))
        out.update(rl_effective=None, rl_in_s_acc=None, rl_first_mismatch=None, rl_first_reject=None, rl_rho=rho,
                   rl_reward=reward, rl_round_return=reward.sum(1))
    return out


def _exact_tree(c, s):
    N = _tree_nodes(c)
    tmax, targ, tlse, tent = _row_stats(s["target"])
    dmax, darg, dlse, dent = _row_stats(s["draft"])
    par, tok = s["parent"].long().clamp(min=0), s["tokens"].long().clamp(min=0)
    inner = torch.zeros(c["B"], N, dtype=torch.bool, device="cuda")
    inner.scatter_(1, par[:, 1:], True)
    nan = torch.full_like(dmax, math.nan)
    root = torch.arange(N, device="cuda") == 0
    lt, ld = nan.clone(), nan.clone()
    for b in range(c["B"]):
        lt[b] = s["target"][b, par[b], tok[b]].double() - tlse[b, par[b]]
        ld[b] = s["draft"][b, par[b], tok[b]].double() - dlse[b, par[b]]
    z = _scores(s["hidden"].reshape(c["B"] * N, -1), s["head"]).reshape(c["B"], N)
    match = root | (tok == targ.gather(1, par))
    zt, pi, acc, la = _verdicts(z, match, c["lam"], None)
    return dict(accept_len=None, tokens=None, path=None, tgt_argmax=None, tgt_max=tmax, tgt_lse=tlse, tgt_entropy=tent,
                drf_argmax=None, drf_max=torch.where(inner, dmax, nan), drf_lse=torch.where(inner, dlse, nan),
                drf_entropy=torch.where(inner, dent, nan), logp_tgt=torch.where(root, nan, lt),
                logp_drf=torch.where(root, nan, ld), delta=None, z_tilde=zt, policy=pi, accept=None,
                tgt_candidate=None, logp_action=la)


def _exact_attention(c, s):
    B, n_q, Hq, D = s["q"].shape
    L, Hkv = s["k"].shape[1], s["k"].shape[2]
    out = torch.zeros(B, n_q, Hq, D, dtype=torch.float64, device="cuda")
    key = torch.arange(L, device="cuda")
    for b in range(B):
        ctx, q0 = int(s["ctx_len"][b]), int(s["q_start"][b])
        n = min(ctx + 2 * c["K"] + 3, L)
        pos = torch.arange(q0, q0 + n_q, device="cuda")
        see = torch.where(pos < ctx, pos + 1, n)
        hide = key[None, :] >= see[:, None]
        for h in range(Hq):
            k = s["k"][b, :, h * Hkv // Hq].double()
            v = s["v"][b, :, h * Hkv // Hq].double().contiguous()
            w = (s["q"][b, :, h].double() @ k.t().contiguous()) * s["scale"]
            o = torch.softmax(w.masked_fill_(hide, -math.inf), -1) @ v
            out[b, :, h] = torch.where((pos < n)[:, None], o, torch.zeros_like(o))
    return out


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "attention":
        return _exact_attention(case, s)
    if kind == "arbitrate":
        return dict(z=_scores(s["hidden"][s["index"].long()], s["head"]), accept=None)
    if kind == "tree":
        return _exact_tree(case, s)
    return _exact_chain(case, s)
