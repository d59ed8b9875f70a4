"""Performance cases of the Fork-dLLM step, as a program that serves or trains
with it calls it: denoising steps over all positions and over the active
blocks, greedy and drawn, in bf16 and fp32; teacher-forced likelihoods; the
unmasking rule alone; the ForkGRPO objective and JustGRPO-Fast's positions.

listed() names them, draw() gives more of the same ranges; prepare() makes a
case's inputs from a seed, run() makes one pass, exact() gives the numbers of
that pass in 64 bits, work() the bytes and operations it cannot do without.
"""
import math

import numpy as np
import torch

from paper_2609_39859_amd import _binding

RULES = {"leftmost": _binding.FORK_RULE_LEFTMOST, "maxconf": _binding.FORK_RULE_MAXCONF,
         "minconf": _binding.FORK_RULE_MINCONF, "maxent": _binding.FORK_RULE_MAXENT,
         "random": _binding.FORK_RULE_RANDOM}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
# most multiply-adds of a drawn case: the largest listed one's (LLaDA-8B
# shape, all rows); fp32 matrix units are about 16 times slower
MOST_MACS = 4096 * 4096 * 126464


def _step(name, B, L, block_len, d, V, dtype="bf16", rows="active", tau=0.9, temperature=0.0,
          rule="leftmost", extras=True):
    c = dict(kind="step", B=B, L=L, block_len=block_len, d=d, V=V, dtype=dtype, rows=rows, tau=tau,
             temperature=temperature, rule=rule, extras=extras)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest model of the test suite, one sequence: launch latency
        _step("step_tiny_f32", 1, 64, 8, 256, 1024, dtype="f32", rows="all", extras=False),
        # a small model, every position scored
        _step("step_mid_all", 4, 256, 32, 1024, 32000, rows="all"),
        # the benchmark's step: LLaDA-8B shape, every position scored
        _step("step_llada8b_all", 8, 512, 32, 4096, 126464, rows="all", extras=False),
        # the same batch served: only the active blocks go through the head
        _step("step_llada8b_active", 8, 512, 32, 4096, 126464),
        # one user's long generation, candidates drawn
        _step("step_single_drawn", 1, 2048, 32, 4096, 126464, temperature=0.8, tau=0.8),
        # ForkGRPO rollouts: 64 sequences at the sampling temperature
        _step("step_rollout_drawn", 64, 384, 32, 4096, 126464, temperature=0.8, tau=0.8),
        # one GPU's share of an 8-way vocabulary split, served
        _step("step_vocab_shard_active", 8, 512, 32, 4096, 15808),
        # sizes that fill no tile: all rows, drawn, highest-entropy fallback
        _step("step_ragged_drawn_all", 3, 301, 20, 1544, 50257, rows="all", tau=0.7,
              temperature=1.0, rule="maxent"),
        # ForkGRPO's likelihoods of one batch's fallback steps
        dict(kind="logprob", name="logprob_batch", n=3847, M=8192, d=4096, V=126464, dtype="bf16"),
        # the rule alone on a large batch of sequences
        dict(kind="select", name="select_large", B=131072, L=64, block_len=32, tau=0.9,
             rule="maxconf", layout="row"),
        # the objective of 16 prompts x 16 rollouts
        dict(kind="grpo", name="grpo_objective", n_groups=16, G=16, per=15),
        # JustGRPO-Fast: the 20% most uncertain positions of 256 rollouts
        dict(kind="top_entropy", name="top_entropy", R=256, Lg=256, k=52),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "logprob", "select", "grpo", "top_entropy"], [6, 2, 1, 1, 1])[0]
    if kind in ("step", "logprob"):
        dtype = rng.choices(["bf16", "f32"], [5, 1])[0]
        d = min(4096, 8 * _log(rng, 16, 512))
        V = _log(rng, 1000, 126464)
        most = MOST_MACS // (1 if dtype == "bf16" else 32) // (d * V)
    if kind == "step":
        B = _log(rng, 1, 64)
        block_len = rng.choice([8, 16, 20, 32, 32, 32, 48, 64])
        L = max(block_len, _log(rng, 64, 2048))
        rows = rng.choice(["all", "active", "active"])
        L = max(block_len, min(L, 65536 // B))
        while B > 1 and B * (L if rows == "all" else block_len) > most:
            B //= 2
        if rows == "all":
            L = max(block_len, min(L, most // B))
        return _step(None, B, L, block_len, d, V, dtype, rows, rng.choice([0.5, 0.8, 0.9, 0.95]),
                     rng.choice([0.0, 0.0, 0.8, 1.0]), rng.choice(list(RULES)),
                     rng.random() < 0.5)
    if kind == "logprob":
        n = max(1, min(_log(rng, 16, 4096), most))
        return dict(kind=kind, n=n, M=n + _log(rng, 1, 4096), d=d, V=V, dtype=dtype)
    if kind == "select":
        block_len = rng.choice([8, 16, 32, 64])
        return dict(kind=kind, B=_log(rng, 16, 131072), L=block_len * rng.randint(1, 4),
                    block_len=block_len, tau=rng.choice([0.5, 0.9]), rule=rng.choice(list(RULES)),
                    layout=rng.choice(["row", "position"]))
    if kind == "grpo":
        return dict(kind=kind, n_groups=_log(rng, 1, 64), G=rng.randint(2, 64),
                    per=_log(rng, 4, 100))
    Lg = _log(rng, 64, 2048)
    return dict(kind=kind, R=_log(rng, 16, 512), Lg=Lg, k=max(1, Lg * rng.randint(5, 50) // 100))


# ------------------------------------------------------------------ inputs

def _head(V, d, dtype, gen, dev):
    """LM-head weights, entries N(0, 1/d)."""
    W = torch.empty(V, d, dtype=DTYPES[dtype], device=dev)
    for v in range(0, V, 16384):
        n = min(16384, V - v)
        W[v:v + n] = torch.randn(n, d, generator=gen, device=dev) / math.sqrt(d)
    return W


def _hidden(M, d, dtype, W, gen, dev):
    """Final hidden states: RMS between 0.5 and 2; 30% of the rows point at
    one vocabulary entry (logit about +20), as confident positions do."""
    h = torch.randn(M, d, generator=gen, device=dev)
    h *= 0.5 + 1.5 * torch.rand(M, 1, generator=gen, device=dev)
    sure = torch.rand(M, 1, generator=gen, device=dev) < 0.3
    v = torch.randint(0, W.shape[0], (M,), generator=gen, device=dev)
    h += torch.where(sure, 20.0, 0.0) * W[v].float()
    return h.to(DTYPES[dtype])


def _decode_state(B, L, block_len, gen):
    """Sequences in the middle of a decode: a prompt, finished blocks, a block
    with some positions left, masked blocks after it; every 16th is done.
    Host arrays (mask [B, L], block_start [B])."""
    prompt = L // 4
    nblocks = max(1, -(-(L - prompt) // block_len))
    mask = np.zeros((B, L), np.uint8)
    start = np.zeros(B, np.int32)
    for b in range(B):
        j = gen.integers(0, nblocks)
        s = min(prompt + j * block_len, L - 1)
        start[b] = s
        if b % 16 == 15:
            continue
        e = min(s + block_len, L)
        mask[b, s:e] = gen.random(e - s) < 0.6
        mask[b, gen.integers(s, e)] = 1
        mask[b, e:] = 1
    return mask, start


def _state_buffer(tokens, mask, start, dev):
    """tokens, block starts and mask in one buffer, so that a request's state
    is restored with one copy: (buffer, tokens, mask, block_start) views."""
    M, B = tokens.size, start.size
    raw = np.concatenate([tokens.astype(np.int32).view(np.uint8).ravel(),
                          start.astype(np.int32).view(np.uint8), mask.ravel()])
    buf = torch.from_numpy(raw).to(dev)
    return (buf, buf[:4 * M].view(torch.int32), buf[4 * (M + B):],
            buf[4 * M:4 * (M + B)].view(torch.int32))


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    host = np.random.default_rng(seed)
    return {"step": _prepare_step, "logprob": _prepare_logprob, "select": _prepare_select,
            "grpo": _prepare_grpo, "top_entropy": _prepare_top}[case["kind"]](case, gen, host, dev)


def _prepare_step(c, gen, host, dev):
    B, L, d, V, BL = c["B"], c["L"], c["d"], c["V"], c["block_len"]
    M = B * L
    W = _head(V, d, c["dtype"], gen, dev)
    h = _hidden(M, d, c["dtype"], W, gen, dev)
    mask, start = _decode_state(B, L, BL, host)
    tokens = np.where(mask.ravel(), -1, host.integers(0, V, M))
    buf, tok, msk, bs = _state_buffer(tokens, mask, start, dev)
    f = {k: torch.zeros(M, device=dev) for k in ("conf", "entropy", "logp")}
    out = dict(f, fallback=torch.zeros(B, dtype=torch.int32, device=dev), tokens=tok, mask=msk,
               block_start=bs)
    kw = dict(B=B, L=L, rule=RULES[c["rule"]], temperature=c["temperature"], seed=20240607,
              counter=17, rows_mode=_binding.FORK_ROWS_ACTIVE if c["rows"] == "active"
              else _binding.FORK_ROWS_ALL)
    if c["rule"] == "random":
        kw["fallback_uniform"] = torch.rand(B, generator=gen, device=dev)
    if c["extras"]:
        out["lse"] = torch.zeros(M, device=dev)
        out["argmax"] = torch.zeros(M, dtype=torch.int32, device=dev)
        out["ncommit"] = torch.zeros(B, dtype=torch.int32, device=dev)
        out["commit_pos"] = torch.zeros(B * BL, dtype=torch.int32, device=dev)
        kw.update(out_lse=out["lse"], out_argmax=out["argmax"], out_ncommit=out["ncommit"],
                  out_commit_pos=out["commit_pos"])
    return dict(kind="step", W=W, h=h, buf=buf, initial=buf.clone(), out=out, kw=kw, BL=BL,
                tau=c["tau"])


def _prepare_logprob(c, gen, host, dev):
    n, M = c["n"], c["M"]
    W = _head(c["V"], c["d"], c["dtype"], gen, dev)
    h = _hidden(M, c["d"], c["dtype"], W, gen, dev)
    rows = torch.randperm(M, generator=gen, device=dev)[:n].sort().values.to(torch.int32)
    toks = torch.randint(0, c["V"], (n,), generator=gen, device=dev, dtype=torch.int32)
    out = {k: torch.zeros(n, device=dev) for k in ("logp", "q", "entropy", "lse")}
    return dict(kind="logprob", W=W, h=h, rows=rows, toks=toks, out=out)


def _prepare_select(c, gen, host, dev):
    B, L, BL = c["B"], c["L"], c["block_len"]
    M = B * L
    # one confident position in 20; the candidate of each position
    conf = torch.rand(B, L, generator=gen, device=dev) * 0.4
    conf += 0.6 * (torch.rand(B, L, generator=gen, device=dev) < 0.05)
    ent = 8.0 * torch.rand(B, L, generator=gen, device=dev)
    cand = torch.randint(0, 126464, (B, L), generator=gen, device=dev, dtype=torch.int32)
    j = torch.randint(0, L // BL, (B, 1), generator=gen, device=dev)
    pos = torch.arange(L, device=dev)
    left = torch.rand(B, L, generator=gen, device=dev) < 0.6
    mask = ((pos >= (j + 1) * BL) | ((pos >= j * BL) & left)).to(torch.uint8)
    mask[torch.arange(B, device=dev), (j * BL).squeeze(1)] = 1
    position = c["layout"] == "position"
    conf, ent, cand, mask = ((x.t() if position else x).contiguous().reshape(M)
                             for x in (conf, ent, cand, mask))
    start = (j * BL).squeeze(1).to(torch.int32).contiguous()
    out = dict(tokens=torch.zeros(M, dtype=torch.int32, device=dev), mask=mask.clone(),
               block_start=start.clone(), fallback=torch.zeros(B, dtype=torch.int32, device=dev),
               ncommit=torch.zeros(B, dtype=torch.int32, device=dev))
    kw = dict(B=B, L=L, rule=RULES[c["rule"]], out_ncommit=out["ncommit"],
              layout=_binding.FORK_LAYOUT_POSITION_MAJOR if position
              else _binding.FORK_LAYOUT_ROW_MAJOR)
    if c["rule"] == "maxent":
        kw["entropy"] = ent
    if c["rule"] == "random":
        kw["uniform"] = torch.rand(B, generator=gen, device=dev)
    return dict(kind="select", conf=conf, cand=cand, mask=mask, out=out, kw=kw, BL=BL, tau=c["tau"])


def _prepare_grpo(c, gen, host, dev):
    ng, G = c["n_groups"], c["G"]
    R = ng * G
    # uneven rollouts, a few of them without a fallback step
    share = host.random(R) * (host.random(R) > 0.05) + 1e-9
    counts = host.multinomial(c["per"] * R, share / share.sum())
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    n = int(off[-1])
    old = -8.0 * torch.rand(n, generator=gen, device=dev)
    new = old + 0.2 * torch.randn(n, generator=gen, device=dev)
    rewards = (torch.rand(R, generator=gen, device=dev) < 0.5).float()
    f = dict(device=dev)
    out = dict(adv=torch.zeros(R, **f), ratio=torch.zeros(n, **f), term=torch.zeros(n, **f),
               rollout_obj=torch.zeros(R, **f), group_obj=torch.zeros(ng, **f),
               skipped=torch.zeros(ng, dtype=torch.uint8, **f), J=torch.zeros(1, **f))
    return dict(kind="grpo", rewards=rewards, offsets=torch.from_numpy(off).to(dev), new=new,
                old=old, G=G, out=out)


def _prepare_top(c, gen, host, dev):
    # entropies of a rollout: mostly near zero, a long tail; some equal
    e = torch.rand(c["R"], c["Lg"], generator=gen, device=dev)
    e = 6.0 * e.pow(4)
    e = torch.where(e < 0.01, torch.zeros_like(e), e)
    return dict(kind="top_entropy", entropy=e, k=c["k"],
                sel=torch.zeros(c["R"], c["Lg"], dtype=torch.uint8, device=dev))


# ---------------------------------------------------------------- one pass

def run(s):
    kind, o = s["kind"], s.get("out")
    if kind == "step":
        s["buf"].copy_(s["initial"])  # the request's state before the step
        _binding.fork_step_ex(s["h"], s["W"], o["tokens"], o["mask"], o["block_start"], s["BL"],
                              s["tau"], o["conf"], o["entropy"], o["logp"], o["fallback"],
                              **s["kw"])
        return o
    if kind == "logprob":
        _binding.logprob(s["h"], s["W"], s["toks"], o["logp"], rows=s["rows"], out_q=o["q"],
                         out_entropy=o["entropy"], out_lse=o["lse"])
        return o
    if kind == "select":
        o["mask"].copy_(s["mask"])
        _binding.select(s["conf"], s["cand"], o["tokens"], o["mask"], o["block_start"], s["BL"],
                        s["tau"], o["fallback"], **s["kw"])
        return o
    if kind == "grpo":
        _binding.grpo_objective(s["rewards"], s["offsets"], s["new"], s["old"], s["G"], 0.2,
                                o["group_obj"], o["skipped"], o["J"], out_adv=o["adv"],
                                out_ratio=o["ratio"], out_term=o["term"],
                                out_rollout_obj=o["rollout_obj"])
        return o
    _binding.top_entropy(s["entropy"], s["k"], s["sel"])
    return s["sel"]


# ------------------------------------------------- what a pass cannot avoid

def work(c):
    k = c["kind"]
    if k in ("step", "logprob"):
        size = 2 if c["dtype"] == "bf16" else 4
        if k == "step":
            M = c["B"] * (c["L"] if c["rows"] == "all" else c["block_len"])
            small = 21 * M + 12 * c["B"]
        else:
            M, small = c["n"], 24 * c["n"]
        return {"bytes": size * c["d"] * (c["V"] + M) + small, "flops": 2.0 * M * c["d"] * c["V"]}
    if k == "select":
        # per sequence: the block's mask bytes and confidences (entropies
        # where they decide), a committed candidate, token, mask byte, flags
        per = 5 * c["block_len"] + (4 * c["block_len"] if c["rule"] == "maxent" else 0) + 25
        return {"bytes": per * c["B"], "flops": 0}
    if k == "grpo":
        R = c["n_groups"] * c["G"]
        return {"bytes": 16 * c["per"] * R + 16 * R + 5 * c["n_groups"], "flops": 0}
    return {"bytes": 5 * c["R"] * c["Lg"], "flops": 0}


def tolerance(c):
    if c["kind"] in ("select", "top_entropy"):
        return "exact"
    if c["kind"] == "grpo":
        return {"rel": 1e-5, "max": 1e-4}
    # fp32 sums of d products: up to 2.2e-6 seen against 64 bits (q of given
    # tokens); a candidate may change where two logits agree to rounding
    return {"rel": 1e-5, "max": 2e-4, "differ": 2e-3}


# -------------------------------------------------------------- in 64 bits

def _stats64(h, W):
    """Per row of h: log-normaliser, entropy and largest logit's log q."""
    W = W.double()
    lse, ent, logp = [], [], []
    rows = max(1, (1 << 28) // W.shape[0])
    for r in range(0, h.shape[0], rows):
        z = h[r:r + rows].double() @ W.t()
        l = torch.logsumexp(z, dim=1)
        lse.append(l)
        logp.append(z.max(dim=1).values - l)
        p = torch.exp(z - l[:, None])
        ent.append(l - (p * z).sum(dim=1))
    return torch.cat(lse), torch.cat(ent), torch.cat(logp)


def exact(case, seed):
    k = case["kind"]
    if k in ("select", "top_entropy"):
        return None
    s = prepare(case, seed)
    o = s["out"]
    if k == "step":
        B, L, BL = case["B"], case["L"], case["block_len"]
        if case["rows"] == "all":
            rows = torch.arange(B * L)
        else:
            mask, start = o["mask"].cpu().view(B, L), o["block_start"].cpu()
            rows = []
            for b in range(B):
                p = int(start[b])
                while p < L and not bool(mask[b, p:p + BL].any()):
                    p += BL
                rows += [b * L + i for i in range(p, min(p + BL, L))]
            rows = torch.tensor(rows, dtype=torch.int64)
        rows = rows.to(s["h"].device)
        lse, ent, logp = _stats64(s["h"][rows], s["W"])

        def at(x):
            return torch.zeros(B * L, dtype=torch.float64, device=x.device).index_copy_(0, rows, x)

        got = dict.fromkeys(o)
        got["entropy"] = at(ent)
        if "lse" in o:
            got["lse"] = at(lse)
        if case["temperature"] == 0.0:  # else they are those of the drawn candidates
            got["conf"], got["logp"] = at(torch.exp(logp)), at(logp)
        return got
    if k == "logprob":
        h = s["h"][s["rows"].long()]
        lse, ent, _ = _stats64(h, s["W"])
        z = (h.double() * s["W"][s["toks"].long()].double()).sum(dim=1)
        return dict(logp=z - lse, q=torch.exp(z - lse), entropy=ent, lse=lse)
    ng, G = case["n_groups"], case["G"]
    r = s["rewards"].double().view(ng, G)
    mean = r.mean(dim=1, keepdim=True)
    sd = (r - mean).square().mean(dim=1, keepdim=True).sqrt()
    adv = torch.where(sd > 0, (r - mean) / sd, torch.zeros_like(r)).view(-1)
    off = s["offsets"].long()
    count = off[1:] - off[:-1]
    owner = torch.repeat_interleave(torch.arange(ng * G, device=off.device), count)
    ratio = torch.exp(s["new"].double() - s["old"].double())
    term = torch.minimum(ratio * adv[owner], ratio.clamp(0.8, 1.2) * adv[owner])
    obj = torch.zeros(ng * G, dtype=torch.float64, device=off.device).index_add_(0, owner, term)
    obj = obj / count.clamp(min=1)
    kept = sd.view(-1) > 0
    group = torch.where(kept, obj.view(ng, G).mean(dim=1), torch.zeros_like(sd.view(-1)))
    J = group.sum() / kept.sum().clamp(min=1)
    return dict(adv=adv, ratio=ratio, term=term, rollout_obj=obj, group_obj=group, skipped=None,
                J=J.view(1))
