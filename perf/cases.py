"""The work that a serving engine has the verification step and the drafter do.

Five kinds of pass, each through the package's public binding with the buffers and workspaces
that an engine keeps from step to step:

  step    one whole verification step: schedule, verify attention, acceptance
  sched   the scheduler alone, Algorithm 1 or its asynchronous form
  attn    ragged paged verify attention (GQA, small heads and pages, fp32, absorbed latent)
  accept  speculative acceptance over the vocabulary (greedy, stochastic, with the analytic rate)
  draft   the drafter's sequential block (Markov or RNN head)

Decisions (accepted lengths, drawn tokens) are kept away from ties: uniforms lie inside the bucket
that they pick, so every correct implementation gives the same whole numbers.
"""
import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2607_05147_amd import dspark

DEV = "cuda"


def listed():
    return [
        # the smallest step an engine makes: four chats, a small fp32 model; launches and latency count
        dict(name="step_tiny", kind="step", R=4, K=8, tokens=29, Hq=8, Hkv=2, Dqk=64, Dv=64, page=16, dt="f32", layout="hnd",
             lo=32, hi=128, median=0, V=1024, logit="f32", mode="greedy"),
        # the asynchronous scheduler at 512 concurrent requests: capacity from an earlier step, then admission
        dict(name="sched_async_highconc", kind="sched", R=512, K=8, knee=512, a=2.0, b=1.0, mode="async"),
        # a few interactive users with long prompts: the batch alone does not fill the chip
        dict(name="attn_interactive", kind="attn", R=4, K=16, tokens=30, Hq=64, Hkv=8, Dqk=128, Dv=128, page=64, dt="bf16",
             layout="hnd", lo=2048, hi=16384, median=0),
        # the headline: 128 requests, grouped-query heads, log-normal contexts
        dict(name="attn_serving", kind="attn", R=128, K=16, tokens=565, Hq=64, Hkv=8, Dqk=128, Dv=128, page=64, dt="bf16",
             layout="hnd", lo=2048, hi=16384, median=4096),
        # an engine with 16-token pages, token-major, and heads of 64
        dict(name="attn_small_pages", kind="attn", R=64, K=8, tokens=190, Hq=32, Hkv=8, Dqk=64, Dv=64, page=16, dt="bf16",
             layout="nhd", lo=512, hi=4096, median=0),
        # a model that is served in fp32
        dict(name="attn_fp32", kind="attn", R=16, K=16, tokens=70, Hq=32, Hkv=8, Dqk=128, Dv=128, page=64, dt="f32",
             layout="hnd", lo=512, hi=2048, median=0),
        # long contexts on an absorbed latent head: 128 query heads on one 576/512 row
        dict(name="attn_latent", kind="attn", R=16, K=16, tokens=77, Hq=128, Hkv=1, Dqk=576, Dv=512, page=64, dt="bf16",
             layout="hnd", lo=32768, hi=131072, median=0),
        # rejection sampling over a large vocabulary at 128 requests
        dict(name="accept_serving", kind="accept", R=128, K=16, tokens=565, V=129280, logit="bf16", mode="stochastic"),
        # fp32 logits, with the analytic acceptance rate that trains the confidence head
        dict(name="accept_mid_rate", kind="accept", R=32, K=16, tokens=140, V=32768, logit="f32", mode="rate"),
        # greedy matching at 512 requests, one to three rows each
        dict(name="accept_greedy", kind="accept", R=512, K=8, tokens=1020, V=129280, logit="bf16", mode="greedy"),
        # the draft block that feeds the serving step
        dict(name="draft_markov", kind="draft", head="markov", R=128, K=16, V=129280, rank=256, d=4096, base="bf16"),
        # the RNN head on a mid-sized model with fp32 base logits
        dict(name="draft_rnn", kind="draft", head="rnn", R=32, K=16, V=32768, rank=256, d=4096, base="f32"),
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng, lo, hi):
    """Vocabularies as models have them: often padded to 64, sometimes to 8, sometimes odd."""
    v = _logu(rng, lo, hi)
    return max(64, v - v % rng.choice([1, 1, 8, 64, 64]))


def draw(rng):
    kind = rng.choice(["step", "sched", "attn", "attn", "attn", "attn", "accept", "accept", "draft", "draft"])
    if kind == "sched":
        K = rng.randint(4, 16)
        R = _logu(rng, 16, min(512, 8192 // K))
        return dict(kind=kind, R=R, K=K, knee=_logu(rng, R, 4 * R + 1), a=rng.choice([2.0, 3.0, 4.0]), b=rng.choice([1.0, 1.5]),
                    mode=rng.choice(["stop", "async"]))
    if kind == "accept":
        K, V = rng.randint(1, 16), _vocab(rng, 1000, 131072)
        R = _logu(rng, 1, 512)
        mode = rng.choice(["stochastic", "stochastic", "rate", "greedy"])
        if mode != "greedy":
            R = max(1, min(R, 270_000_000 // (K * V)))
        tokens = min(R * (K + 1), R + int(R * K * rng.uniform(0.1, 0.6)), max(R, 140_000_000 // V))
        return dict(kind=kind, R=R, K=K, tokens=tokens, V=V, logit=rng.choice(["bf16", "f32"]), mode=mode)
    if kind == "draft":
        K, V = rng.randint(2, 16), _vocab(rng, 2000, 131072)
        R = max(1, min(_logu(rng, 1, 200), 260_000_000 // (K * V)))
        return dict(kind=kind, head=rng.choice(["markov", "rnn"]), R=R, K=K, V=V, rank=rng.choice([64, 128, 256]),
                    d=rng.choice([0, 520, 1024, 2048, 4096]), base=rng.choice(["bf16", "f32"]))
    K = rng.randint(1, 16)
    if kind == "step":
        R = _logu(rng, 1, 48)
        tokens = R + int(R * K * rng.uniform(0.1, 0.6))
        shape = rng.choice([dict(Hq=8, Hkv=2, Dqk=64, Dv=64, page=16, dt="f32"), dict(Hq=32, Hkv=8, Dqk=128, Dv=128, page=64, dt="bf16"),
                            dict(Hq=16, Hkv=8, Dqk=128, Dv=128, page=16, dt="bf16")])
        lo = _logu(rng, 32, 1024)
        V = _vocab(rng, 1000, 40000)
        return dict(kind=kind, R=R, K=K, tokens=tokens, layout=rng.choice(["hnd", "nhd"]), lo=max(lo, K + 1), hi=lo + _logu(rng, 32, 2048),
                    median=0, V=V, logit=rng.choice(["bf16", "f32"]), mode=rng.choice(["greedy", "stochastic"]), **shape)
    family = rng.choice(["gqa", "gqa", "small", "small", "f32", "latent"])
    layout = rng.choice(["hnd", "nhd"])
    if family == "latent":
        R, lo = _logu(rng, 1, 32), _logu(rng, 256, 65536)
        hi = lo + _logu(rng, 64, 65536)
        Hq, rate = rng.choice([16, 64, 128]), rng.uniform(0.1, 0.6)
        R = max(1, min(R, int(300_000_000 / ((lo + hi) / 2 * Hq * (1 + K * rate) * 0.6))))
        return dict(kind=kind, R=R, K=K, tokens=R + int(R * K * rate), Hq=Hq, Hkv=1, Dqk=576, Dv=512, page=rng.choice([16, 64]) if R <= 4 and hi <= 8192 else 64,
                    dt="bf16", layout="hnd", lo=lo, hi=hi, median=0)
    R, rate = _logu(rng, 1, 256), rng.uniform(0.1, 0.6)
    lo = _logu(rng, 64, 8192)
    hi = lo + _logu(rng, 64, 8192)
    Hkv, group = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 5, 8])
    if family == "gqa":
        D, Dv, page, dt = 128, 128, rng.choice([64, 64, 128, 256]), "bf16"
    elif family == "small":
        D, Dv = rng.choice([(64, 64), (64, 64), (80, 80), (96, 96), (128, 128), (192, 128), (256, 256)])
        page, dt = rng.choice([16, 16, 32, 48, 64]), "bf16"
    else:
        (D, Dv), page, dt = rng.choice([(64, 64), (128, 128)]), rng.choice([16, 32, 64]), "f32"
    most = 4_000_000 if family == "gqa" else 1_000_000 if family == "small" else 300_000
    R = max(1, min(R, int(most / ((lo + hi) / 2 * Hkv) * 128 / D)))
    return dict(kind=kind, R=R, K=K, tokens=R + int(R * K * rate), Hq=Hkv * group, Hkv=Hkv, Dqk=D, Dv=Dv, page=page, dt=dt,
                layout=layout, lo=max(lo, K + 1), hi=hi, median=0)


# ------------------------------------------------------------------ inputs

_T = {"f32": torch.float32, "bf16": torch.bfloat16}


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 64 + stream)
    return g


def _randn(seed, stream, *shape, dtype=torch.float32, scale=1.0):
    x = torch.randn(*shape, generator=_gen(seed, stream), device=DEV, dtype=dtype)
    return x.mul_(scale) if scale != 1.0 else x


def _confidences(R, K, a, b, seed, stream):
    return np.random.default_rng([seed, stream]).beta(a, b, (R, K)).astype(np.float32)


def _lengths(c, seed):
    """Verification lengths as the scheduler gives them: the most likely drafts, `tokens` rows in all."""
    R, K = c["R"], c["K"]
    surv = np.cumprod(_confidences(R, K, 4.0, 1.5, seed, 1).astype(np.float64), axis=1)
    admit = np.zeros(R * K, bool)
    admit[np.argsort(-surv.ravel(), kind="stable")[: min(R * K, c["tokens"] - R)]] = True
    return admit.reshape(R, K).sum(1).astype(np.int32)


def _context_quantiles(c, u):
    if c["median"]:
        z = np.array([NormalDist().inv_cdf(float(x)) for x in u])
        return np.clip(c["median"] * np.exp(0.5 * z), c["lo"], c["hi"])
    return c["lo"] + u * (c["hi"] - c["lo"])


def _contexts(c, seed):
    u = np.random.default_rng([seed, 2]).uniform(1e-6, 1 - 1e-6, c["R"])
    return np.rint(_context_quantiles(c, u)).astype(np.int64)


def _mean_context(c):
    return float(_context_quantiles(c, (np.arange(2000) + 0.5) / 2000).mean())


def _attention_inputs(c, seed, lens):
    """Query rows, the paged cache in shuffled pages and what addresses it."""
    R, Hkv, page, dt = c["R"], c["Hkv"], c["page"], _T[c["dt"]]
    kv = np.maximum(_contexts(c, seed), lens + 1)
    pages = (kv + page - 1) // page
    max_pages, total = int(pages.max()), int(pages.sum())
    perm = np.random.default_rng([seed, 3]).permutation(total).astype(np.int32)
    table = np.zeros((R, max_pages), np.int32)
    at = 0
    for r in range(R):
        table[r, : pages[r]] = perm[at : at + pages[r]]
        at += int(pages[r])

    def cache(stream, D):
        strides = (Hkv * page * D, page * D, D) if c["layout"] == "hnd" else (page * Hkv * D, D, Hkv * D)
        return _randn(seed, stream, total * Hkv * page * D, dtype=dt), strides

    k, ks = cache(4, c["Dqk"])
    v, vs = (k, ks) if c["Dqk"] == 576 else cache(5, c["Dv"])
    rows = R * (c["K"] + 1)  # the engine's buffers hold the largest batch
    return dict(q=_randn(seed, 6, rows, c["Hq"], c["Dqk"], dtype=dt), k=k, v=v, ks=ks, vs=vs, table=torch.from_numpy(table).to(DEV),
                kv_len=torch.from_numpy(kv.astype(np.int32)).to(DEV), out=torch.zeros(rows, c["Hq"], c["Dv"], dtype=dt, device=DEV),
                attn_ws=torch.empty(max(256, dspark.dspark_verify_attn_workspace_size(R, c["K"] + 1, c["Hq"], Hkv, c["Dqk"], c["Dv"], max_pages, page, dt)),
                                    dtype=torch.uint8, device=DEV))


def _accept_inputs(c, seed, lens):
    """Target logits of the verified rows, drafts, and uniforms away from ties."""
    R, K, V, dt = c["R"], c["K"], c["V"], _T[c["logit"]]
    cu = np.concatenate([[0], np.cumsum(lens + 1)]).astype(np.int64)
    logits = _randn(seed, 7, int(cu[-1]), V, scale=4.0).to(dt)
    s = dict(logits=logits, draft_p=None, u=None, rate=None, accepted=torch.zeros(R, dtype=torch.int32, device=DEV),
             token=torch.zeros(R, dtype=torch.int32, device=DEV),
             accept_ws=torch.empty(dspark.dspark_accept_workspace_size(R, K, V), dtype=torch.uint8, device=DEV))
    rng = np.random.default_rng([seed, 8])
    tok = rng.integers(0, V, (R, K))
    if c["mode"] == "greedy":
        best = logits.float().argmax(1).cpu().numpy()
        hit = rng.random((R, K)) < 0.7
        for r in range(R):
            n = int(lens[r])
            tok[r, :n] = np.where(hit[r, :n], best[cu[r] : cu[r] + n], tok[r, :n])
        s["tok"] = torch.from_numpy(tok.astype(np.int32)).to(DEV)
        return s
    # draft distributions: the target at temperature 0.8, mixed 80/20 with a sparse perturbation
    draft_p = torch.zeros(R, K, V, device=DEV)
    g = _gen(seed, 9)
    u = rng.random((R, K + 1)).astype(np.float32)
    for r in range(R):
        n = int(lens[r])
        pt = torch.softmax(logits[cu[r] : cu[r + 1]].double(), 1)
        accepted = n
        if n:
            noise = torch.rand(n, V, generator=g, device=DEV).pow_(12.0)
            pd = 0.8 * torch.softmax(logits[cu[r] : cu[r] + n].float() / 0.8, 1) + 0.2 * noise / noise.sum(1, keepdim=True)
            draft_p[r, :n] = pd
            x = torch.multinomial(pd, 1, generator=g)
            ratio = (pt[:n].gather(1, x) / pd.double().gather(1, x)).squeeze(1).cpu().numpy()
            tok[r, :n] = x.squeeze(1).cpu().numpy()
            near = np.abs(u[r, :n] - ratio) < 2e-3
            u[r, :n] = np.where(near, np.where(u[r, :n] < 0.5, u[r, :n] + 0.01, u[r, :n] - 0.01), u[r, :n])
            passed = u[r, :n] < ratio
            accepted = n if passed.all() else int(np.argmin(passed))
        mass = pt[accepted] if accepted == n else (pt[accepted] - draft_p[r, accepted].double()).clamp_(min=0)
        _, u[r, K] = _inside(mass[None], u[r : r + 1, K])
    s["tok"] = torch.from_numpy(tok.astype(np.int32)).to(DEV)
    s["draft_p"], s["u"] = draft_p, torch.from_numpy(u).to(DEV)
    if c["mode"] == "rate":
        s["rate"] = torch.zeros(int(cu[-1]), device=DEV)
    return s


def _inside(mass, u):
    """The tokens that uniforms u [n] draw from mass [n, V] (fp64, device), among those with a mass over 2e-5 of
    the row, and a uniform inside each one's bucket."""
    cum = mass.cumsum(1)
    total = cum[:, -1:]
    sure = torch.where(mass > 2e-5 * total, mass, torch.zeros_like(mass)).cumsum(1)
    at = torch.from_numpy(np.asarray(u, np.float64)).to(DEV)[:, None] * sure[:, -1:]
    x = torch.searchsorted(sure, at, right=True).clamp_(max=mass.shape[1] - 1)
    share = 0.25 + 0.5 * torch.from_numpy(np.asarray(u, np.float64)).to(DEV)[:, None]
    inside = (cum.gather(1, x) - (1 - share) * mass.gather(1, x)) / total
    return x.squeeze(1), inside.squeeze(1).float().cpu().numpy()


def _draft64(c, s, pick):
    """The draft block in 64 bits. pick(k, p): the tokens of position k from p [R, V]. Returns tokens, p (per position) and conf."""
    R, K, rank, d = c["R"], c["K"], c["rank"], c["d"]
    w2 = s["W2t"].double().t().contiguous()
    state = torch.zeros(R, rank, dtype=torch.float64, device=DEV)
    wc = s["w_conf"].double()
    x, toks, ps, confs = s["anchor"].long(), [], [], []
    base = s["base"].view(R, K, c["V"])
    for k in range(K):
        e = s["W1"][x].double()
        h = s["hidden"][:, k].double() if d else None
        bias = e
        if c["head"] == "rnn":
            a = torch.cat([state, e] + ([h] if d else []), 1) @ s["Wrnn"].double().t()
            gate = torch.sigmoid(a[:, :rank])
            state = gate * state + (1 - gate) * torch.tanh(a[:, rank : 2 * rank])
            bias = torch.tanh(a[:, 2 * rank :])
        p = torch.softmax(base[:, k].double() + bias @ w2, 1)
        logit = e @ wc[d:] + (h @ wc[:d] if d else 0.0)
        confs.append(torch.sigmoid(logit / s["temp"][k].double()))
        x = pick(k, p)
        toks.append(x)
        ps.append(p)
    return torch.stack(toks, 1), ps, torch.stack(confs, 1)


def _draft_inputs(c, seed):
    R, K, V, rank, d = c["R"], c["K"], c["V"], c["rank"], c["d"]
    bf = torch.bfloat16
    s = dict(anchor=torch.randint(0, V, (R,), generator=_gen(seed, 10), device=DEV, dtype=torch.int32),
             base=_randn(seed, 11, R * K, V, scale=4.0).to(_T[c["base"]]),
             W1=_randn(seed, 12, V, rank, scale=rank ** -0.5).to(bf), W2t=_randn(seed, 13, V, rank).to(bf),
             hidden=_randn(seed, 14, R, K, d).to(bf) if d else None, w_conf=_randn(seed, 15, d + rank, scale=(d + rank) ** -0.5),
             temp=1.0 + 0.05 * torch.arange(1, K + 1, device=DEV, dtype=torch.float32))
    size = dspark.dspark_markov_draft_workspace_size
    if c["head"] == "rnn":
        size = dspark.dspark_rnn_draft_workspace_size
        scale = torch.cat([torch.full((rank,), rank ** -0.5), torch.ones(rank), torch.full((d,), max(d, 1) ** -0.5)]).to(DEV)
        w = _randn(seed, 16, 3 * rank, 2 * rank + d) * scale
        w[2 * rank :] *= rank ** -0.5
        s["Wrnn"] = w.to(bf)
    u = np.random.default_rng([seed, 17]).random((R, K)).astype(np.float32)

    def pick(k, p):
        x, u[:, k] = _inside(p, u[:, k])
        return x

    _draft64(c, s, pick)
    s.update(u=torch.from_numpy(u).to(DEV), tok=torch.zeros(R, K, dtype=torch.int32, device=DEV), p=torch.zeros(R, K, V, device=DEV),
             conf=torch.zeros(R, K, device=DEV), ws=torch.empty(size(R, K, V, rank), dtype=torch.uint8, device=DEV))
    return s


def _sched_inputs(c, seed):
    R, K = c["R"], c["K"]
    t = np.arange(R * (K + 1) + 1, dtype=np.float64)
    sps = 1.0 / (1.0 + np.maximum(0.0, t - c["knee"]) / 1024.0)
    dev = lambda x: torch.from_numpy(x).to(DEV)  # noqa: E731
    i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=DEV)  # noqa: E731
    return dict(conf=dev(_confidences(R, K, c["a"], c["b"], seed, 18)), prev=dev(_confidences(R, K, c["a"], c["b"], seed, 19)), sps=dev(sps),
                len=i32(R), cu=i32(R + 1), tok_req=i32(R * (K + 1)), cap=i32(1),
                sched_ws=torch.empty(dspark.dspark_schedule_workspace_size(R, K), dtype=torch.uint8, device=DEV))


def prepare(case, seed):
    c = case
    s = dict(c=c, max_q=c["K"] + 1)
    if c["kind"] == "sched":
        s.update(_sched_inputs(c, seed))
        return s
    if c["kind"] == "draft":
        s.update(_draft_inputs(c, seed))
        return s
    lens = _lengths(c, seed)
    if c["kind"] == "step":
        # the scheduler's own lengths: its capacity is the batch that the engine asked for
        s.update(_sched_inputs(dict(R=c["R"], K=c["K"], knee=c["tokens"], a=4.0, b=1.5), seed))
        s["conf"] = torch.from_numpy(_confidences(c["R"], c["K"], 4.0, 1.5, seed, 1)).to(DEV)
        s["cap"].fill_(c["tokens"] - c["R"])
    else:
        s["cu"] = torch.from_numpy(np.concatenate([[0], np.cumsum(lens + 1)]).astype(np.int32)).to(DEV)
    if c["kind"] in ("step", "attn"):
        s.update(_attention_inputs(c, seed, lens))
    if c["kind"] in ("step", "accept"):
        s.update(_accept_inputs(c, seed, lens))
    return s


# ------------------------------------------------------------------ one pass

def _attend(s):
    c = s["c"]
    out, _ = dspark.dspark_verify_attn(s["q"], s["k"], s["v"], s["ks"], s["vs"], s["table"], s["kv_len"], s["cu"], s["max_q"], c["Hkv"],
                                       c["Dv"], c["page"], c["Dqk"] ** -0.5, out=s["out"], ws=s["attn_ws"])
    return out


def _accept(s):
    acc, tok, rate = dspark.dspark_accept(s["tok"], s["logits"], s["cu"], draft_p=s["draft_p"], u=s["u"], accepted_len=s["accepted"],
                                          next_tok=s["token"], accept_rate=s["rate"], ws=s["accept_ws"])
    return dict(accepted=acc, token=tok) if rate is None else dict(accepted=acc, token=tok, rate=rate)


def run(state):
    s = state
    c = s["c"]
    kind = c["kind"]
    if kind == "attn":
        return dict(out=_attend(s))
    if kind == "accept":
        return _accept(s)
    if kind == "step":
        dspark.dspark_schedule_topk(s["conf"], s["cap"], s["len"], s["cu"], s["tok_req"], ws=s["sched_ws"])
        return dict(len=s["len"], cu=s["cu"], out=_attend(s), **_accept(s))
    if kind == "sched":
        if c["mode"] == "stop":
            dspark.dspark_schedule(s["conf"], s["sps"], 0, s["len"], s["cu"], s["tok_req"], ws=s["sched_ws"])
            return dict(len=s["len"], cu=s["cu"], tok_req=s["tok_req"])
        dspark.dspark_schedule_capacity(s["prev"], s["sps"], s["cap"], ws=s["sched_ws"])
        dspark.dspark_schedule_topk(s["conf"], s["cap"], s["len"], s["cu"], s["tok_req"], ws=s["sched_ws"])
        return dict(cap=s["cap"], len=s["len"], cu=s["cu"], tok_req=s["tok_req"])
    more = dict(hidden=s["hidden"], sts_temp=s["temp"], draft_tok=s["tok"], draft_p=s["p"], conf=s["conf"], ws=s["ws"])
    if c["head"] == "markov":
        tok, p, conf = dspark.dspark_markov_draft(s["anchor"], s["base"], s["W1"], s["W2t"], s["w_conf"], s["u"], c["K"], **more)
    else:
        tok, p, conf = dspark.dspark_rnn_draft(s["anchor"], s["base"], s["W1"], s["W2t"], s["Wrnn"], s["w_conf"], s["u"], c["K"], **more)
    return dict(tok=tok, p=p, conf=conf)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    c = case
    R, K = c["R"], c["K"]
    size = {"f32": 4, "bf16": 2}
    n = f = 0.0
    if c["kind"] in ("sched", "step"):
        twice = 2 if c.get("mode") == "async" else 1
        n += twice * (R * K * 4 + 8 * (R * (K + 1) + 1)) + 4 * (2 * R + 1 + R * (K + 1))
        f += twice * R * K
    if c["kind"] in ("attn", "step"):
        kv, e = _mean_context(c), size[c["dt"]]
        per_key = c["Dqk"] if c["Dqk"] == 576 else c["Dqk"] + c["Dv"]  # latent values are the key rows
        n += R * kv * c["Hkv"] * per_key * e + c["tokens"] * c["Hq"] * (c["Dqk"] + c["Dv"]) * e + R * 4 * kv / c["page"]
        f += 2.0 * c["tokens"] * kv * c["Hq"] * (c["Dqk"] + c["Dv"])
    if c["kind"] in ("accept", "step"):
        drafts = {"greedy": 0, "stochastic": 0.6 * R, "rate": c["tokens"] - R}[c["mode"]]  # rows of draft_p: of the rejections, or all tested
        n += c["tokens"] * c["V"] * size[c["logit"]] + drafts * c["V"] * 4
        f += 4.0 * c["tokens"] * c["V"]
    if c["kind"] == "draft":
        V, rank, d = c["V"], c["rank"], c["d"]
        # base logits and p of every row; the projection once for the block; hidden states; embeddings
        n += R * K * V * (size[c["base"]] + 4) + V * rank * 2 + R * K * (d * 2 + rank * 2)
        f += 2.0 * R * K * V * rank
        if c["head"] == "rnn":
            n += 3 * rank * (2 * rank + d) * 2
            f += 2.0 * R * K * 3 * rank * (2 * rank + d)
    return {"bytes": n, "flops": f}


def tolerance(case):
    # against exact(), the path shows 2.3e-3 (bf16 attention, its output's rounding), 6e-7 (fp32 attention), 6e-8 (the rate),
    # 5e-7 (p, Markov head) and 2.3e-6 (p, RNN head, whose output enters its product as two bf16 terms)
    kind = case["kind"]
    if kind == "attn" or kind == "step":
        return {"rel": 1e-2, "max": 0.1} if case["dt"] == "bf16" else {"rel": 3e-6, "max": 4e-5}
    if kind == "accept" and case["mode"] == "rate":
        return {"rel": 1e-6, "max": 4e-5}
    if kind == "draft":
        return {"rel": 4e-6, "max": 2e-4} if case["head"] == "markov" else {"rel": 1.5e-5, "max": 6e-4}
    return "exact"


# ------------------------------------------------------------------ the same in 64 bits

def _exact_attention(c, s, lens):
    R, Hkv, page, group = c["R"], c["Hkv"], c["page"], c["Hq"] // c["Hkv"]
    out = torch.zeros(R * (c["K"] + 1), c["Hq"], c["Dv"], dtype=torch.float64, device=DEV)
    table, kv_len = s["table"].long(), s["kv_len"].cpu().tolist()
    at = 0

    def rows(cache, r, kv, D):
        hnd = c["layout"] == "hnd"
        pages = cache.view(-1, Hkv, page, D) if hnd else cache.view(-1, page, Hkv, D).transpose(1, 2)
        x = pages[table[r, : (kv + page - 1) // page]]
        return x.transpose(0, 1).reshape(Hkv, -1, D)[:, :kv].double()

    for r in range(R):
        ql, kv = int(lens[r]) + 1, kv_len[r]
        k, v = rows(s["k"], r, kv, c["Dqk"]), rows(s["v"], r, kv, c["Dqk"] if c["Dqk"] == 576 else c["Dv"])[..., : c["Dv"]]
        mask = torch.arange(kv, device=DEV)[None] > kv - ql + torch.arange(ql, device=DEV)[:, None]
        for g in range(Hkv):
            q = s["q"][at : at + ql, g * group : (g + 1) * group].double().transpose(0, 1)  # group, ql, D
            z = (q.reshape(-1, c["Dqk"]) @ k[g].t()).view(group, ql, kv).mul_(c["Dqk"] ** -0.5).masked_fill_(mask, -math.inf)
            o = torch.softmax(z, -1).reshape(-1, kv) @ v[g]
            out[at : at + ql, g * group : (g + 1) * group] = o.view(group, ql, c["Dv"]).transpose(0, 1)
        at += ql
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "sched" or c["kind"] == "accept" and c["mode"] != "rate":
        return None  # whole numbers only
    if c["kind"] == "draft":
        s = prepare(c, seed)
        u = s["u"].double()
        tok, ps, conf = _draft64(c, s, lambda k, p: torch.searchsorted(p.cumsum(1), u[:, k : k + 1], right=True).clamp_(max=c["V"] - 1).squeeze(1))
        return dict(tok=None, p=torch.stack(ps, 1), conf=conf)
    s = prepare(c, seed)
    lens = _lengths(c, seed)
    if c["kind"] == "accept":
        rate, at = torch.full((c["tokens"],), -1.0, dtype=torch.float64, device=DEV), 0
        for r in range(c["R"]):
            n = int(lens[r])
            pt = torch.softmax(s["logits"][at : at + n].double(), 1)
            rate[at : at + n] = torch.minimum(pt, s["draft_p"][r, :n].double()).sum(1)
            at += n + 1
        return dict(accepted=None, token=None, rate=rate)
    out = _exact_attention(c, s, lens)
    return dict(out=out) if c["kind"] == "attn" else dict(len=None, cu=None, out=out, accepted=None, token=None)
