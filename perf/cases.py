"""Timed cases of the re-scoring library, through its public entry points.

A case is one call (or one short chain of calls) that a training program makes
with this library: scoring sampled tokens under one or both contexts, picking
branch points, building groups, and the gradients of a token-level loss
through the lm-head.  Sizes are those of the repository's own workloads
(`workloads/synth.py`, `bench.py`) or generic ones between them.

Kinds of cases, and the ranges that `draw` covers:

  rescore   both contexts of R roots of T positions, then the k branch points
            of every root.  2 R T = 32 .. 524,288 rows, d 256 .. 5120 (any
            multiple of 8), V 4,096 .. 152,064; bf16, or fp32 up to 4,096 rows,
            d 1024 and V 50,257; all positions, a prefix excluded, or
            tool-observation spans excluded
  logprobs  log p and log-sum-exp of n = 16 .. 65,536 rows (same d, V, dtypes)
  noalloc   the same without a workspace, into the caller's buffers
  entropy   log p and next-token entropy of R roots under the original
            context, then the k positions of highest entropy
  backward  dL/dhidden and dL/dW of n = 64 .. 32,768 rows (bf16)
  update    log p, the clipped policy loss's per-token factor, then backward
  select    the k branch points of R = 1 .. 512 roots of T = 64 .. 40,000
            positions from given log p pairs, with the signed difference
  group     constrained selection, continuation slots, advantages and loss
            factors of 4 .. 128 problems with trajectories of 256 .. 8192 tokens
"""
import math

import numpy as np
import torch

import paper_2609_36864_amd as hdl

MAX_DRAWN_FLOPS = 6e13


def listed():
    return [
        # the repository's small fp32 workload: one root, both contexts; every launch and the call's host work count
        dict(name="rescore_tiny_f32", kind="rescore", R=1, T=256, d=256, V=4096, dtype="f32", mask="all", k=4),
        # one short answer scored under one context, as a serving loop does between rollouts: into its own buffers
        dict(name="noalloc_short", kind="noalloc", n=96, d=2048, V=151936, dtype="bf16", mask="none"),
        # a single root re-scored when it finishes: both contexts, the prompt's end excluded, an odd length
        dict(name="rescore_one_root", kind="rescore", R=1, T=777, d=4096, V=151936, dtype="bf16", mask="prefix", k=2),
        # ragged everything: a K tail (d is no multiple of 64), an odd vocabulary, observation spans
        dict(name="logprobs_ragged", kind="logprobs", n=3333, d=1000, V=50257, dtype="bf16", mask="spans"),
        # fp32 hidden states and weights, a small model's sizes
        dict(name="logprobs_f32", kind="logprobs", n=2048, d=1024, V=32000, dtype="f32", mask="none"),
        # the Entropy selector over a few roots (original context only)
        dict(name="entropy_two_roots", kind="entropy", R=2, T=4096, d=2048, V=151936, dtype="bf16", mask="prefix", k=8),
        # math roots: 8 x 2 x 4096, the middle workload
        dict(name="rescore_math", kind="rescore", R=8, T=4096, d=2048, V=151936, dtype="bf16", mask="prefix", k=8),
        # agent roots with observation spans: 32 x 2 x 8192, the benchmark's workload and the largest call
        dict(name="rescore_agent", kind="rescore", R=32, T=8192, d=4096, V=151936, dtype="bf16", mask="spans", k=8),
        # one short trajectory's training step: scoring, loss factor and both gradients
        dict(name="update_short", kind="update", n=300, d=2048, V=151936, dtype="bf16", mask="prefix"),
        # gradients of a whole micro-batch (the benchmark's backward pass)
        dict(name="backward_math", kind="backward", n=32768, d=2048, V=151936, dtype="bf16", mask="prefix"),
        # branch points of a few long roots
        dict(name="select_long", kind="select", R=4, T=32768, k=32, mask="spans"),
        # group construction of one training step at the paper's batch
        dict(name="group_batch", kind="group", problems=128, T=4096),
    ]


# ---- drawn cases -----------------------------------------------------------

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _model(rng, dtype):
    """(d, V) of a drawn case."""
    if dtype == "f32":
        return 8 * _log_int(rng, 16, 128), _log_int(rng, 1000, 50257)
    d = rng.choice((1024, 2048, 2560, 4096, 5120)) if rng.random() < 0.5 else 8 * _log_int(rng, 32, 640)
    v = rng.choice((32000, 50257, 151936, 152064)) if rng.random() < 0.6 else _log_int(rng, 4096, 152064)
    return d, v


def _cap_rows(n, d, v, per_row=2.0):
    return max(16, min(n, int(MAX_DRAWN_FLOPS / (per_row * d * v))))


def draw(rng):
    kind = rng.choice(("rescore", "rescore", "logprobs", "noalloc", "entropy", "backward", "update", "select", "group"))
    mask = rng.choice(("all", "prefix", "spans"))
    if kind == "select":
        R, T = _log_int(rng, 1, 512), _log_int(rng, 64, 40000)
        return dict(kind=kind, R=R, T=T, k=min(T, _log_int(rng, 1, 64)), mask=mask)
    if kind == "group":
        return dict(kind=kind, problems=_log_int(rng, 4, 128), T=_log_int(rng, 256, 8192))
    dtype = "f32" if kind in ("rescore", "logprobs") and rng.random() < 0.25 else "bf16"
    d, V = _model(rng, dtype)
    if kind in ("rescore", "entropy"):
        per = 4.0 if kind == "rescore" else 2.0   # flops per position / (d V)
        rows = _cap_rows(_log_int(rng, 32, 4096 if dtype == "f32" else 524288), d, V)
        T = max(16, min(32768, int(rows / per * 2.0 ** rng.uniform(-4, 0))))
        R = max(1, int(rows / (per / 2.0) / T))
        return dict(kind=kind, R=R, T=T, d=d, V=V, dtype=dtype, mask=mask, k=min(8, max(1, T // 16)))
    if kind in ("backward", "update"):
        n = _cap_rows(_log_int(rng, 64, 32768), d, V, 8.0)
        return dict(kind=kind, n=n, d=d, V=V, dtype="bf16", mask=mask)
    n = _cap_rows(_log_int(rng, 16, 4096 if dtype == "f32" else 65536), d, V)
    return dict(kind=kind, n=n, d=d, V=V, dtype=dtype, mask=rng.choice(("none", mask)))


# ---- inputs ----------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _mask(kind, R, T, seed):
    """[R, T] uint8 on the GPU (None for "none"): 1 where the policy wrote the token."""
    if kind == "none":
        return None
    m = np.ones((R, T), np.uint8)
    rs = np.random.RandomState(seed % (1 << 31))
    if kind == "prefix":
        m[:, :min(32, T // 8)] = 0
    elif kind == "spans":
        for r in range(R):
            for _ in range(rs.randint(5, 21)):
                ln = min(int(rs.randint(64, 513)), max(1, T // 16))
                st = int(rs.randint(0, T - ln + 1))
                m[r, st:st + ln] = 0
    return torch.from_numpy(m).cuda()


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _weight(case, g):
    w = torch.empty(case["V"], case["d"], dtype=_dtype(case), device="cuda")
    for v in range(0, case["V"], 32768):
        n = min(32768, case["V"] - v)
        w[v:v + n] = torch.randn(n, case["d"], device="cuda", generator=g) * 0.02
    return w


def _rows(n, d, g):
    x = torch.randn(n, d, device="cuda", generator=g)
    return x / x.square().mean(1, keepdim=True).sqrt()


def _spread(n, lo, hi, g):
    """n values spread over [lo, hi] in a random order, no two close together."""
    step = (hi - lo) / n
    x = lo + step * (torch.arange(n, device="cuda") + 0.25 + 0.5 * torch.rand(n, device="cuda", generator=g))
    return x[torch.randperm(n, device="cuda", generator=g)]


def _planted(mask, r, T, n, g):
    """Up to n eligible positions of root r."""
    elig = torch.arange(T, device="cuda") if mask is None else torch.nonzero(mask[r]).view(-1)
    return elig[torch.randperm(elig.numel(), device="cuda", generator=g)[:n]]


def _rescore_inputs(case, seed):
    R, T, d, k = case["R"], case["T"], case["d"], case["k"]
    g = _gen(seed)
    w = _weight(case, g)
    mask = _mask(case["mask"], R, T, seed)
    tokens = torch.randint(0, case["V"], (R, T), device="cuda", generator=g, dtype=torch.int32)
    hidden = torch.empty(2, R, T, d, dtype=w.dtype, device="cuda")
    for r in range(R):
        h0 = _rows(T, d, g).to(w.dtype)
        hidden[0, r] = h0
        h1 = h0.float() + 0.01 * torch.randn(T, d, device="cuda", generator=g)
        # positions whose sampled token the hindsight context moves by 0.5 to 5 nats
        pos = _planted(mask, r, T, k + 8, g)
        wy = w[tokens[r, pos].long()].float()
        a = _spread(pos.numel(), 0.5, 5.0, g)
        a = torch.where(torch.rand(pos.numel(), device="cuda", generator=g) < 0.5, -a, a)
        h1[pos] += a[:, None] * wy / wy.square().sum(1, keepdim=True)
        hidden[1, r] = h1.to(w.dtype)
    return dict(hidden=hidden, w=w, tokens=tokens, mask=mask)


def _entropy_inputs(case, seed):
    R, T, k = case["R"], case["T"], case["k"]
    g = _gen(seed)
    w = _weight(case, g)
    mask = _mask(case["mask"], R, T, seed)
    tokens = torch.randint(0, case["V"], (R * T,), device="cuda", generator=g, dtype=torch.int32)
    hidden = torch.empty(R * T, case["d"], dtype=w.dtype, device="cuda")
    for r in range(R):
        # most positions are decided, a few are open to different degrees
        temp = 1.5 + 1.5 * torch.rand(T, device="cuda", generator=g)
        pos = _planted(mask, r, T, k + 8, g)
        temp[pos] = _spread(pos.numel(), 0.3, 1.2, g)
        hidden[r * T:(r + 1) * T] = _rows(T, case["d"], g) * temp[:, None]
    return dict(hidden=hidden, w=w, tokens=tokens, mask=mask)


def _row_inputs(case, seed):
    n = case["n"]
    g = _gen(seed)
    w = _weight(case, g)
    mask = _mask(case["mask"], 1, n, seed)
    hidden = torch.empty(n, case["d"], dtype=w.dtype, device="cuda")
    for i in range(0, n, 16384):
        m = min(16384, n - i)
        hidden[i:i + m] = _rows(m, case["d"], g)
    tokens = torch.randint(0, case["V"], (n,), device="cuda", generator=g, dtype=torch.int32)
    s = dict(hidden=hidden, w=w, tokens=tokens, mask=None if mask is None else mask.view(-1))
    if case["kind"] == "noalloc":
        s["logp"] = torch.empty(n, device="cuda")
        s["lse"] = torch.empty(n, device="cuda")
    elif case["kind"] == "backward":
        # upstream gradients of the token-level loss; lse as the forward pass left it
        s["g"] = torch.randn(n, device="cuda", generator=g) / n
        s["lse"] = _exact_stats(hidden, w, tokens)[1].float()
    elif case["kind"] == "update":
        # trajectories of up to 512 tokens; the rollout's log p differs a little from the current one
        n_traj = -(-n // 512)
        s["traj"] = (torch.arange(n, device="cuda") // 512).to(torch.int32)
        s["adv"] = torch.randn(n_traj, device="cuda", generator=g)
        s["logp_old"] = _exact_stats(hidden, w, tokens)[0].float() + 0.2 * torch.randn(n, device="cuda", generator=g)
    return s


def _pairs(R, T, g):
    lo = torch.empty(R, T, device="cuda").exponential_(1.0 / 3.0, generator=g).neg_() - 1e-3
    return lo, torch.clamp(lo + 0.5 * torch.randn(R, T, device="cuda", generator=g), max=0.0)


def _group_inputs(case, seed):
    n_groups, roots, alloc, T = case["problems"], 2, (3, 4), case["T"]
    g = _gen(seed)
    R = n_groups * roots
    lo, hi = _pairs(R, T, g)
    n_traj = n_groups * roots * (1 + sum(alloc))
    old = torch.empty(n_traj * T, device="cuda").exponential_(0.5, generator=g).neg_()
    edge = min(32, T // 8)
    return dict(
        n_groups=n_groups, roots=roots, alloc=alloc, lo=lo, hi=hi, mask=_mask("spans", R, T, seed),
        rlo=torch.full((R,), edge, dtype=torch.int32, device="cuda"),
        rhi=torch.full((R,), T - 1 - edge, dtype=torch.int32, device="cuda"),
        rewards=(torch.rand(n_groups, n_traj // n_groups, device="cuda", generator=g) < 0.5).float(),
        traj=torch.arange(n_traj, dtype=torch.int32, device="cuda").repeat_interleave(T),
        pos=torch.arange(T, dtype=torch.int32, device="cuda").repeat(n_traj), logp_old=old,
        logp_new=old + 0.2 * torch.randn(n_traj * T, device="cuda", generator=g),
        loss_mask=(torch.rand(n_traj * T, device="cuda", generator=g) < 0.9).to(torch.uint8),
        start=torch.zeros(n_traj, dtype=torch.int32, device="cuda"),
        n_trained=torch.zeros(1, dtype=torch.int64, device="cuda"))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "rescore":
        s = _rescore_inputs(case, seed)
    elif kind == "entropy":
        s = _entropy_inputs(case, seed)
    elif kind == "select":
        lo, hi = _pairs(case["R"], case["T"], _gen(seed))
        s = dict(lo=lo, hi=hi, mask=_mask(case["mask"], case["R"], case["T"], seed))
    elif kind == "group":
        s = _group_inputs(case, seed)
    else:
        s = _row_inputs(case, seed)
    s.update(kind=kind, k=case.get("k"), R=case.get("R"), T=case.get("T"))
    return s


# ---- one pass --------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "rescore":
        return hdl.rescore(s["hidden"], s["w"], s["tokens"], s["mask"], s["k"])
    if kind == "logprobs":
        return hdl.token_logprobs(s["hidden"], s["w"], s["tokens"], s["mask"])
    if kind == "noalloc":
        hdl.token_logprobs_noalloc(s["hidden"], s["w"], s["tokens"], s["mask"], s["logp"], s["lse"])
        return s["logp"], s["lse"]
    if kind == "entropy":
        mask = s["mask"].view(-1)
        logp, lse, ent = hdl.token_logprobs(s["hidden"], s["w"], s["tokens"], mask, want_entropy=True)
        idx, score, count = hdl.select_top_k(ent.view(s["R"], s["T"]), s["mask"], s["k"])
        return logp, lse, ent, idx, score, count
    if kind == "backward":
        return hdl.token_logprobs_backward(s["hidden"], s["w"], s["tokens"], s["mask"], s["lse"], s["g"])
    if kind == "update":
        logp, lse = hdl.token_logprobs(s["hidden"], s["w"], s["tokens"], s["mask"])
        g, loss = hdl.policy_loss_grad(s["adv"], s["traj"], logp, s["logp_old"], loss_mask=s["mask"])
        dh, dw = hdl.token_logprobs_backward(s["hidden"], s["w"], s["tokens"], s["mask"], lse, g)
        return logp, loss, dh, dw
    if kind == "select":
        return hdl.select_branch_points(s["lo"], s["hi"], s["mask"], s["k"], want_delta=True)
    idx, score, count = hdl.select_constrained(s["lo"], s["hi"], s["mask"], len(s["alloc"]), lo=s["rlo"], hi=s["rhi"],
                                               min_gap=64)
    bpos, rank = hdl.allocate_continuations(idx, count, s["alloc"])
    # a problem's roots, then their continuations, each trained from its branch position on
    s["start"].view(s["n_groups"], -1)[:, s["roots"]:] = bpos.view(s["n_groups"], -1)
    adv = hdl.group_advantages(s["rewards"])
    g, loss = hdl.policy_loss_grad(adv.view(-1), s["traj"], s["logp_new"], s["logp_old"], loss_mask=s["loss_mask"],
                                   pos=s["pos"], start=s["start"], n_trained=s["n_trained"])
    return idx, score, count, bpos, rank, adv, g, loss


# ---- what a pass cannot do without -------------------------------------------

def _share(case, n):
    """About how many of n rows a mask leaves (spans: 12.5 spans of at most T / 16)."""
    if case["mask"] == "spans":
        T = case.get("T") or case["n"]
        return n * math.exp(-12.5 * min(288.0, T / 16.0) / T)
    if case["mask"] == "prefix":
        T = case.get("T") or case["n"]
        return n * (1.0 - min(32, T // 8) / T)
    return n


def work(case):
    kind = case["kind"]
    if kind == "select":
        n = case["R"] * case["T"]
        return {"bytes": n * (8 + 1 + 4) + case["R"] * (8 * case["k"] + 4), "flops": 2 * n}
    if kind == "group":
        R, n = 2 * case["problems"], 16 * case["problems"] * case["T"]
        return {"bytes": R * case["T"] * 9 + n * 25, "flops": 12 * n}
    rows = case["n"] if "n" in case else case["R"] * case["T"] * (2 if kind == "rescore" else 1)
    scored = _share(case, rows)
    d, V, esz = case["d"], case["V"], 4 if case["dtype"] == "f32" else 2
    b = V * d * esz + scored * d * esz + rows * 13
    f = 2.0 * scored * d * V
    if kind == "backward":
        return {"bytes": b + 4 * (V * d + rows * d), "flops": 3 * f}
    if kind == "update":   # scoring keeps no logits: recomputed once for the gradient
        return {"bytes": b + 4 * (V * d + rows * d), "flops": 4 * f}
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind == "select":
        return "exact"   # one fp32 subtraction; ranks and ties are defined
    if kind == "group":
        return {"rel": 1e-6, "max": 1e-4}   # 4.7e-8 off the 64-bit result
    if kind in ("backward", "update"):
        return {"rel": 7e-3}   # the logit gradient is rounded to bf16: 1.7e-3 off the 64-bit result
    # fp32 sums over d, then over the vocabulary: at most 2.8e-7 off the 64-bit result
    return {"rel": 1.2e-6, "max": 5e-5}


# ---- 64-bit results ----------------------------------------------------------

def _exact_stats(hidden, w, tokens, entropy=False):
    """(log p, lse, entropy or None) of every row in float64."""
    n, V = hidden.shape[0], w.shape[0]
    logp = torch.empty(n, dtype=torch.float64, device="cuda")
    lse = torch.empty_like(logp)
    ent = torch.empty_like(logp) if entropy else None
    wd = w.double()
    step = max(1, min(n, (1 << 29) // V))
    for i in range(0, n, step):
        z = hidden[i:i + step].double() @ wd.t()
        l = torch.logsumexp(z, 1)
        logp[i:i + step] = z.gather(1, tokens[i:i + step].long()[:, None]).view(-1) - l
        lse[i:i + step] = l
        if entropy:
            z -= l[:, None]
            ent[i:i + step] = -(z.exp() * z).sum(1)
    return logp, lse, ent


def _exact_grads(hidden, w, tokens, lse, g):
    n, V = hidden.shape[0], w.shape[0]
    wd, hd = w.double(), hidden.double()
    dh = torch.empty_like(hd)
    dw = torch.zeros_like(wd)
    step = max(1, min(n, (1 << 29) // V))
    for i in range(0, n, step):
        p = (hd[i:i + step] @ wd.t() - lse[i:i + step, None]).exp_()
        gi = g[i:i + step, None]
        p.mul_(-gi).scatter_add_(1, tokens[i:i + step].long()[:, None], gi)
        dh[i:i + step] = p @ wd
        dw += p.t() @ hd[i:i + step]
    return dh, dw


def _on(mask, n):
    return torch.ones(n, device="cuda", dtype=torch.bool) if mask is None else mask.view(-1) != 0


def _top(values, mask, k):
    """Scores of the k best eligible positions of every root, in order, 0 where there are fewer."""
    v = values.clone()
    if mask is not None:
        v[mask == 0] = -math.inf
    top = torch.topk(v, min(k, v.shape[1]), dim=1).values
    top = torch.nn.functional.pad(top, (0, k - top.shape[1]), value=-math.inf)
    return torch.where(torch.isfinite(top), top, torch.zeros_like(top))


def _exact_policy(adv, traj, new, old, on):
    """(g, loss) of the clipped loss, token-level mean over the tokens that are on."""
    a = adv.double()[traj.long()]
    r = torch.exp(new.double() - old.double())
    cut = r.clamp(1 - 0.2, 1 + 0.28)
    scale = 1.0 / max(1, int(on.sum()))
    zero = torch.zeros_like(r)
    g = torch.where(on & (r * a <= cut * a), -a * r * scale, zero)
    return g, torch.where(on, -torch.minimum(r * a, cut * a) * scale, zero)


def _exact_group(s):
    R, T = s["lo"].shape
    score = (s["hi"] - s["lo"]).abs()   # the score is one fp32 subtraction
    t = torch.arange(T, device="cuda")
    fine = (s["mask"] != 0) & (t >= s["rlo"][:, None]) & (t <= s["rhi"][:, None])
    v = torch.where(fine, score.double(), torch.full((), -math.inf, dtype=torch.float64, device="cuda"))
    top, at = (x.cpu().numpy() for x in torch.sort(v, dim=1, descending=True, stable=True))
    out, bpos = np.zeros((R, 2)), np.zeros((R, 7), np.int64)
    for r in range(R):
        kept = []
        for j in range(2):
            if math.isfinite(top[r, j]) and all(abs(at[r, j] - at[r, i]) >= 64 for i in kept):
                kept.append(j)
        out[r, :len(kept)] = top[r, kept]
        first = at[r, kept[0]] if kept else 0
        bpos[r] = [first] * 3 + [at[r, kept[1]] if len(kept) > 1 else first] * 4
    adv = s["rewards"].double()
    adv = adv - adv.mean(1, keepdim=True)
    start = torch.zeros(s["n_groups"], 16, dtype=torch.int64, device="cuda")
    start[:, 2:] = torch.from_numpy(bpos).cuda().view(s["n_groups"], 14)
    on = (s["loss_mask"] != 0) & (s["pos"] >= start.view(-1)[s["traj"].long()])
    # the clip decision is taken on the fp32 ratio's side of the bound; tokens on the bound are rare
    g, loss = _exact_policy(adv.view(-1), s["traj"], s["logp_new"], s["logp_old"], on)
    return None, torch.from_numpy(out), None, None, None, adv, g, loss


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("select", "group") and work(case)["flops"] > 1.5e14:
        return None
    s = prepare(case, seed)
    if kind == "select":
        return None, _top((s["hi"] - s["lo"]).abs().double(), s["mask"], case["k"]), None, None
    if kind == "group":
        return _exact_group(s)
    if kind == "rescore":
        R, T = case["R"], case["T"]
        tok = s["tokens"].view(-1).repeat(2)
        logp = _exact_stats(s["hidden"].view(2 * R * T, -1), s["w"], tok)[0]
        logp[~_on(None if s["mask"] is None else s["mask"].view(-1).repeat(2), 2 * R * T)] = 0
        lp = logp.view(2, R, T)
        return lp, None, _top((lp[1] - lp[0]).abs(), s["mask"], case["k"]), None
    on = _on(s["mask"], s["hidden"].shape[0])
    if kind == "backward":
        return _exact_grads(s["hidden"], s["w"], s["tokens"], s["lse"].double(), torch.where(on, s["g"].double(), 0.0))
    logp, lse, ent = _exact_stats(s["hidden"], s["w"], s["tokens"], kind == "entropy")
    for x in (logp, ent) if kind == "entropy" else (logp,):
        x[~on] = 0
    if kind == "update":
        g, loss = _exact_policy(s["adv"], s["traj"], logp, s["logp_old"], on)
        return (logp, loss) + _exact_grads(s["hidden"], s["w"], s["tokens"], lse, g)
    lse[~on] = 0
    if kind == "entropy":
        return logp, lse, ent, None, _top(ent.view(case["R"], case["T"]), s["mask"], case["k"]), None
    return logp, lse
