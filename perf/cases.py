"""The calls this library exists for, as measurable cases.

Four kinds of pass, each through the public entry points of
paper_2608_20375_amd:

round   one decoding round of a batch: Context.build_tree on fresh drafter
        logits (with or without hidden states, fixed or SABA budgets), then
        Context.accept against the target model's tokens.  This is what a
        serving loop calls once per decoding step, so most cases are rounds,
        from one sequence over a 32000-word vocabulary to 128 sequences of
        32 positions over 151936 words.
verify  what follows a round on the verifier's side: Context.mask_to_bias
        (before the target model's forward pass), Context.accept with a target
        per node, Context.commit_accepted of the accepted path's key/value rows.
train   one TdesTrainer.step: objective, gradient and AdamW of the edge scorer.
fit     one saba_fit: SABA's parameters from a same-prefix replay log.

Inputs are drawn on the GPU from the seed alone; exact() repeats the same
draws and computes the results in 64 bits with torch and numpy only.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_20375_amd as G

HIST_WINDOW = 4


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # One sequence, short block, small vocabulary, small fixed tree: the
        # smallest call, where launches and latency count.
        dict(name="round_b1_v32k_k4", kind="round", batch=1, L=8, V=32000, K=4, N=32, E=64, m=16,
             mode="literal", budget=32, temper=False, hidden=0),
        # One sequence on a 151936-word vocabulary: single-user serving.
        dict(name="round_b1_v152k_k8", kind="round", batch=1, L=16, V=151936, K=8, N=64, E=64,
             m=16, mode="literal", budget=64, temper=False, hidden=0),
        # Sixteen sequences with SABA budgets and the drafter's hidden states
        # (degeneration signal): a small serving batch with the full state.
        dict(name="round_b16_k8_hidden", kind="round", batch=16, L=16, V=151936, K=8, N=256, E=64,
             m=16, mode="paper", budget=0, temper=False, hidden=4096),
        # A ragged round: odd vocabulary (misaligned rows), K and m that fill no
        # tile, few sequences, N not a multiple of 64.
        dict(name="round_b5_ragged_k13", kind="round", batch=5, L=12, V=70001, K=13, N=100, E=60,
             m=20, mode="paper", budget=0, temper=True, hidden=0),
        # The batch-64 serving round of the headline benchmark.
        dict(name="round_b64_k16", kind="round", batch=64, L=16, V=128256, K=16, N=512, E=128,
             m=32, mode="literal", budget=0, temper=True, hidden=0),
        # The largest block and candidate set supported: long drafts, wide trees.
        dict(name="round_b8_L64_k64", kind="round", batch=8, L=64, V=151936, K=64, N=1024, E=128,
             m=64, mode="paper", budget=0, temper=True, hidden=0),
        # The largest batch: 128 sequences of 32 positions and 32 candidates.
        dict(name="round_b128_k32", kind="round", batch=128, L=32, V=151936, K=32, N=1024, E=128,
             m=32, mode="literal", budget=0, temper=True, hidden=0),
        # Verifier side of one sequence: fp32 bias, 16-layer cache of 1 KiB rows.
        dict(name="verify_b1_fp32", kind="verify", batch=1, L=16, N=64, planes=32, width=512,
             bias="float32", V=151936),
        # Verifier side of the batch-64 round: bf16 bias, 36 layers of keys and
        # values, 8 heads of 128 dimensions.
        dict(name="verify_b64_bf16", kind="verify", batch=64, L=16, N=512, planes=72, width=1024,
             bias="bfloat16", V=128256),
        # A training step on a small batch of traces, and on the benchmark's.
        dict(name="train_g512_m16", kind="train", groups=512, pairs=512, K=8, E=64, m=16, L=16,
             V=151936),
        dict(name="train_g4096_m32", kind="train", groups=4096, pairs=4096, K=16, E=128, m=32,
             L=16, V=128256),
        # SABA's fit on a log of 20000 replayed rounds over the 32..512 grid.
        dict(name="fit_t20000_b31", kind="fit", rounds=20000, first=32, step=16, count=31),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a round in six of ten draws, then verify, train and fit."""
    u = rng.random()
    if u < 0.6:
        L = rng.choice((_log_int(rng, 4, 64), 8, 16, 16, 32))
        K = rng.choice((_log_int(rng, 2, 64), 4, 8, 16, 32))
        V = rng.choice((_log_int(rng, 8000, 151936), 32000, 128256, 151936))
        m = rng.choice((16, 32, rng.randint(8, 64)))
        most = 128 * 32 * 151936 // (L * V)
        batch = max(1, min(_log_int(rng, 1, 128), most, 4096 // L, 4194304 // (L * K * K)))
        N = _log_int(rng, 24, 1024)
        return dict(kind="round", batch=batch, L=L, V=V, K=K, N=N, E=rng.choice((32, 64, 100, 128)),
                    m=m, mode=rng.choice(("literal", "paper")),
                    budget=N if rng.random() < 0.3 else 0, temper=rng.random() < 0.5,
                    hidden=8 * rng.randint(64, 512) if rng.random() < 0.3 else 0)
    if u < 0.74:
        return dict(kind="verify", batch=_log_int(rng, 1, 64), L=rng.choice((8, 16, 32)),
                    N=_log_int(rng, 24, 512), planes=rng.randint(8, 72),
                    width=8 * rng.randint(16, 128), bias=rng.choice(("float32", "bfloat16")),
                    V=rng.choice((32000, 128256, 151936)))
    if u < 0.88:
        E, m = rng.choice(((32, 64), (64, 16), (64, 40), (128, 16), (128, 32), (128, 20)))
        return dict(kind="train", groups=_log_int(rng, 64, 4096), pairs=_log_int(rng, 64, 4096),
                    K=rng.choice((4, 8, 13, 16)), E=E, m=m, L=rng.choice((8, 12, 16)),
                    V=rng.choice((32000, 128256, 151936)))
    step = rng.choice((8, 16))
    return dict(kind="fit", rounds=_log_int(rng, 200, 20000), first=step * rng.randint(1, 4),
                step=step, count=rng.randint(6, 31))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _budget_grid(N):
    """Ascending budgets up to N: multiples of 16 from 32 on (at most 64 of
    them), or a few sizes where N is small."""
    if N >= 64:
        g = list(range(32, N + 1, 16))
    else:
        g = sorted({max(1, N // 4), max(1, N // 2), N})
    return g[:64]


def _saba(case):
    N = case["N"]
    return dict(budgets=_budget_grid(N), phi=(6.0, 2000.0, 0.5, 18.0 if N <= 512 else 40.0),
                tau_min=1.0, c0=1.0, c1=2.0 / N, c2=2e-7)


def _round_inputs(case, seed):
    g = _gen(seed)
    dev = "cuda"
    B, L, V, K, E, m = (case[k] for k in ("batch", "L", "V", "K", "E", "m"))
    logits = torch.empty(B, L, V, dtype=torch.bfloat16, device=dev)
    nb = min(L, V)                          # boosted ids a row
    wts = 6.0 * torch.arange(1, nb + 1, device=dev, dtype=torch.float32) ** -1.2
    boosted = torch.empty(B, L, 2, dtype=torch.int64, device=dev)
    per = max(1, (1 << 26) // (L * V))
    for b in range(0, B, per):
        n = min(per, B - b)
        z = torch.randn(n, L, V, device=dev, generator=g)
        if case["temper"]:
            z /= torch.empty(n, L, 1, device=dev).uniform_(0.5, 1.5, generator=g)
        # distinct ids: a random start, then random gaps below V / nb
        gap = torch.randint(1, max(2, V // nb), (n, L, nb), device=dev, generator=g)
        start = torch.randint(0, V, (n, L, 1), device=dev, generator=g)
        ids = (start + gap.cumsum(-1)) % V
        perm = torch.rand(n, L, nb, device=dev, generator=g).argsort(-1)
        ids = ids.gather(-1, perm)
        z.scatter_add_(2, ids, wts.expand(n, L, nb))
        logits[b:b + n] = z.to(torch.bfloat16)
        boosted[b:b + n] = ids[:, :, :2] if nb > 1 else ids.expand(n, L, 2)
    i32 = dict(dtype=torch.int32, device=dev)
    prefix = torch.randint(64, 4097, (B,), device=dev, generator=g).to(torch.int32)
    second = (torch.rand(B, L, device=dev, generator=g) < 0.3).long()
    td = torch.empty(B, L + 1, **i32)
    td[:, :L] = boosted.gather(2, second.unsqueeze(-1)).squeeze(-1).to(torch.int32)
    td[:, L] = torch.randint(0, V, (B,), device=dev, generator=g).to(torch.int32)
    d = dict(logits=logits, prefix=prefix, base=prefix - 1, target_depth=td,
             root=torch.randint(0, V, (B,), device=dev, generator=g).to(torch.int32),
             hist=torch.randint(0, 17, (B,), device=dev, generator=g).float(),
             emb=torch.randn(V, E, device=dev, generator=g) * 0.1,
             g_parent=torch.randn(E, m, device=dev, generator=g) * 0.05,
             g_child=torch.randn(E, m, device=dev, generator=g) * 0.05, u=None, hidden=None)
    if case["mode"] == "paper":
        d["u"] = torch.randn(L, m, device=dev, generator=g) * 0.05
        d.update(scale=1.5, beta=0.2, center=1)
    else:
        d.update(scale=float(np.float32(math.sqrt(m))), beta=1.0, center=0)
    d["beta"] = float(np.float32(d["beta"]))
    if case["hidden"]:
        H = case["hidden"]
        ramp = 0.5 + 2.5 * torch.arange(L, device=dev, dtype=torch.float32) / max(L - 1, 1)
        s = torch.empty(B, 1, 1, device=dev).uniform_(0.3, 1.5, generator=g)
        c = torch.randn(B, 1, H, device=dev, generator=g)
        n = torch.randn(B, L, H, device=dev, generator=g)
        d["hidden"] = (s * ramp[None, :, None] * c + n).to(torch.bfloat16)
    return d


def _verify_inputs(case, seed):
    """Random trees in canonical order (breadth first), their masks, a target
    per node that follows the tree four times out of five, and the verifier's
    key/value rows."""
    g = np.random.default_rng([int(seed), case["batch"], case["N"]])
    B, L, N, V = case["batch"], case["L"], case["N"], case["V"]
    W = (N + 63) // 64
    n = g.integers(max(1, N // 2), N + 1, B)
    ratio = g.uniform(0.3, 0.55, B)
    ratio = np.minimum(ratio, float(N) ** (-1.0 / max(1, L - 2)))
    i = np.arange(N)
    par = np.floor(i[None, :] * ratio[:, None]).astype(np.int64) - 1    # non-decreasing, < i
    par[:, 0] = -1
    on = i[None, :] < n[:, None]
    tok = np.cumsum(g.integers(1, max(2, V // N), (B, N)), axis=1) % V
    mask = np.zeros((B, N, W), np.uint64)
    depth = np.zeros((B, N), np.int64)
    rows = np.arange(B)
    for k in range(N):
        p = par[:, k]
        up = p >= 0
        mask[up, k] = mask[rows[up], p[up]]
        mask[:, k, k >> 6] |= np.uint64(1) << np.uint64(k & 63)
        depth[:, k] = np.where(up, depth[rows, np.maximum(p, 0)] + 1, 1)
    assert int(depth.max()) <= L
    mask[~on] = 0
    # target of the root (slot 0) and of every node (slot k + 1): a child's token
    tgt = g.integers(0, V, (B, N + 1))
    follow = g.random((B, N)) < 0.5
    for k in range(N - 1, -1, -1):          # the children written last win: small indices
        w = on[:, k] & (follow[:, k] | (g.random(B) < 0.4))
        tgt[rows[w], par[w, k] + 1] = tok[w, k]
    T = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda").to(t)
    pad = lambda a, v: np.where(on, a, v)
    gen = _gen(seed)
    src = torch.empty(case["planes"], B, N, case["width"], dtype=torch.bfloat16, device="cuda")
    src.view(torch.int16).random_(-16000, 16000, generator=gen)
    return dict(n=n, par=par, tok=tok, on=on, tgt=tgt,
                n_nodes=T(n, torch.int32), tokens=T(pad(tok, -1), torch.int32),
                parents=T(pad(par, -1), torch.int32),
                mask=torch.from_numpy(mask.view(np.int64)).cuda(),
                target_root=T(tgt[:, 0], torch.int32),
                target_node=T(pad(tgt[:, 1:], -1), torch.int32), src=src)


TRAIN_STEP = 100


def _train_inputs(case, seed):
    """Traces shaped like the rounds and a scorer in the middle of its training:
    warm moments, step 100 on."""
    g = _gen(seed)
    dev = "cuda"
    Gn, P, K, E, m, L, V = (case[k] for k in ("groups", "pairs", "K", "E", "m", "L", "V"))
    i32 = torch.int32
    r = lambda lo, hi, *s: torch.randint(lo, hi, s, device=dev, generator=g)
    # token frequencies fall off as in text: the cube of a uniform number
    perm = torch.randperm(V, device=dev, generator=g)
    word = lambda *s: perm[(torch.rand(*s, device=dev, generator=g) ** 3 * V).long().clamp_(max=V - 1)]
    parent = word(Gn)
    child = (word(Gn, 1) + r(1, max(2, V // (K + 1)), Gn, K).cumsum(-1)) % V    # distinct
    depth = 1 + (torch.rand(Gn, device=dev, generator=g) ** 2 * L).long().clamp_(max=L - 1)
    e = torch.empty(Gn, K, device=dev).exponential_(generator=g)
    logq = -0.2 - 0.7 * e.cumsum(-1)
    z = 2.0 * logq + torch.randn(Gn, K, device=dev, generator=g)
    best = child.gather(1, z.argmax(1, keepdim=True)).squeeze(1)
    hit = torch.rand(Gn, device=dev, generator=g) < 0.8
    target = torch.where(hit, best, torch.full_like(best, -1))
    k = r(0, Gn, P)
    alt = child[k, r(0, K, P)]
    wrong_child = torch.rand(P, device=dev, generator=g) < 0.5
    pairs = torch.stack([parent[k], best[k], depth[k],
                         torch.where(wrong_child, parent[k], word(P)),
                         torch.where(wrong_child, alt, best[k]), depth[k]], dim=1)
    n = 2 * E * m + L * m + 1
    theta = torch.randn(n, device=dev, generator=g) * 0.05
    theta[-1] = 1.5
    adam_v = (torch.randn(n, device=dev, generator=g) * 1e-3) ** 2 + 1e-8
    adam_m = torch.randn(n, device=dev, generator=g) * 2e-4
    batch = dict(parent=parent.to(i32), depth=depth.to(i32), child=child.to(i32), logq=logq,
                 z=z, target=target.to(i32), pairs=pairs.to(i32))
    return dict(emb=torch.randn(V, E, device=dev, generator=g) * 0.1, batch=batch, theta=theta,
                adam_m=adam_m, adam_v=adam_v)


FIT_START = (10.0, 20.0, 20.0, 20.0)
FIT_TAU_MIN = 8.0


def _fit_inputs(case, seed):
    g = _gen(seed)
    dev = "cuda"
    T = case["rounds"]
    grid = [case["first"] + case["step"] * j for j in range(case["count"])]
    f64 = dict(dtype=torch.float64, device=dev)
    uni = lambda lo, hi: torch.empty(T, **f64).uniform_(lo, hi, generator=g)
    B = torch.tensor(grid, **f64)
    state = torch.stack([uni(0.2, 0.95), uni(0.6, 1.4), uni(1, 12)], 1)
    prefix = torch.randint(64, 4097, (T,), device=dev, generator=g)
    tau = (6.0 + state @ torch.tensor([40.0, 30.0, 12.0], **f64)).clamp(min=FIT_TAU_MIN)
    A = uni(2, 14)
    noise = lambda: 1.0 + 0.05 * torch.randn(T, len(grid), generator=g, **f64)
    acc = A[:, None] * (1 - torch.exp(-B / tau[:, None])) * noise()
    lat = (20.0 + 0.05 * B + 2e-5 * B * prefix[:, None]) * noise()
    return dict(grid=grid, state=state.float(), prefix=prefix.to(torch.int32),
                accepted=acc.float(), latency=lat.float())


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "round":
        d = _round_inputs(case, seed)
        B, L, V, K, N = (case[k] for k in ("batch", "L", "V", "K", "N"))
        ctx = G.Context(B, L, V, K, N, HIST_WINDOW)
        ctx.set_scorer(d["emb"], d["g_parent"], d["g_child"], d["u"], d["scale"], d["beta"],
                       d["center"])
        fixed = None
        if case["budget"]:
            fixed = torch.full((B,), case["budget"], dtype=torch.int32, device="cuda")
        else:
            ctx.set_saba(**_saba(case))
        i32 = dict(dtype=torch.int32, device="cuda")
        return dict(kind=kind, ctx=ctx, logits=d["logits"], root=d["root"], base=d["base"],
                    prefix=d["prefix"], hist=d["hist"], fixed=fixed, hidden=d["hidden"],
                    target=d["target_depth"],
                    out=G.TreeBuffers(ctx, B, adj_cos=bool(case["hidden"])),
                    acc_len=torch.empty(B, **i32), acc_nodes=torch.empty(B, L, **i32),
                    bonus=torch.empty(B, **i32))
    if kind == "verify":
        d = _verify_inputs(case, seed)
        B, L, N = case["batch"], case["L"], case["N"]
        ctx = G.Context(B, L, case["V"], 8, N, HIST_WINDOW)
        i32 = dict(dtype=torch.int32, device="cuda")
        # rows of the bias start on 16-byte boundaries
        bias = torch.zeros(B, N, (N + 7) // 8 * 8, dtype=getattr(torch, case["bias"]),
                           device="cuda")
        return dict(kind=kind, ctx=ctx, n_nodes=d["n_nodes"], tokens=d["tokens"],
                    parents=d["parents"], mask=d["mask"], target_root=d["target_root"],
                    target_node=d["target_node"], src=d["src"], bias=bias,
                    dst=torch.zeros(case["planes"], B, L, case["width"], dtype=torch.bfloat16,
                                    device="cuda"),
                    acc_len=torch.empty(B, **i32), acc_nodes=torch.empty(B, L, **i32),
                    bonus=torch.empty(B, **i32))
    if kind == "train":
        d = _train_inputs(case, seed)
        tr = G.TdesTrainer(case["V"], case["E"], case["m"], case["L"], case["K"], case["groups"],
                           case["pairs"])
        return dict(kind=kind, trainer=tr, step=TRAIN_STEP,
                    hyper=G.TdesHyper(w1=float(case["K"] - 1)),
                    loss=torch.zeros(4, dtype=torch.float64, device="cuda"),
                    grad=torch.zeros_like(d["theta"]), **d)
    if kind == "fit":
        return dict(kind=kind, **_fit_inputs(case, seed))
    raise ValueError(kind)


def run(s):
    kind = s["kind"]
    if kind == "round":
        o = s["ctx"].build_tree(s["logits"], s["root"], s["base"], prefix_len=s["prefix"],
                                hist=s["hist"], fixed_budget=s["fixed"], hidden=s["hidden"],
                                out=s["out"])
        a = s["ctx"].accept(o.n_nodes, o.tokens, o.parents, target_depth=s["target"],
                            acc_len=s["acc_len"], acc_nodes=s["acc_nodes"], bonus=s["bonus"])
        r = dict(budget=o.budget, n_nodes=o.n_nodes, tokens=o.tokens, parents=o.parents,
                 pos_ids=o.pos_ids, mask=o.mask, topk_ids=o.topk_ids, topk_logq=o.topk_logq,
                 row_lse=o.row_lse, row_maxprob=o.row_maxprob, row_entropy=o.row_entropy,
                 node_scores=o.node_scores, saba_state=o.saba_state, acc_len=a[0],
                 acc_nodes=a[1], bonus=a[2])
        if s["hidden"] is not None:
            r["adj_cos"] = o.adj_cos
        return r
    if kind == "verify":
        ctx = s["ctx"]
        bias = ctx.mask_to_bias(s["n_nodes"], s["mask"], s["bias"])
        a = ctx.accept(s["n_nodes"], s["tokens"], s["parents"], target_root=s["target_root"],
                       target_node=s["target_node"], acc_len=s["acc_len"],
                       acc_nodes=s["acc_nodes"], bonus=s["bonus"])
        dst = ctx.commit_accepted(a[0], a[1], s["src"], s["dst"])
        return dict(bias=bias, acc_len=a[0], acc_nodes=a[1], bonus=a[2], dst=dst)
    if kind == "train":
        s["trainer"].step(s["emb"], s["batch"], s["theta"], s["adam_m"], s["adam_v"], s["step"],
                          s["hyper"], loss=s["loss"], grad=s["grad"])
        s["step"] += 1
        return dict(theta=s["theta"], adam_m=s["adam_m"], adam_v=s["adam_v"], loss=s["loss"],
                    grad=s["grad"])
    f = G.saba_fit(s["grid"], s["state"], s["prefix"], s["accepted"], s["latency"], FIT_TAU_MIN,
                   FIT_START)
    return dict(phi=np.array(f["phi"]), c=np.array(f["c"]),
                sse=np.array([f["gain_sse"], f["cost_sse"]]))


def work(case):
    kind = case["kind"]
    if kind == "round":
        B, L, V, K, N, m = (case[k] for k in ("batch", "L", "V", "K", "N", "m"))
        W = (N + 63) // 64
        read = B * (L * V * 2 + 2 * L * K * m * 4 + L * case["hidden"] * 2 + L * 4)
        wrote = B * (N * (12 + 8 + 8 * W) + L * K * 8 + L * 16 + 40)
        return dict(bytes=read + wrote, flops=B * L * (V * 5 + K * K * 2 * m))
    if kind == "verify":
        B, L, N = case["batch"], case["L"], case["N"]
        W = (N + 63) // 64
        es = 2 if case["bias"] == "bfloat16" else 4
        # the accepted path is about three nodes long
        return dict(bytes=B * (N * N * es + N * W * 8 + N * 12 + L * 4)
                    + 2 * 3 * B * case["planes"] * case["width"] * 2, flops=B * N * N)
    if kind == "train":
        Gn, P, K, E, m, L = (case[k] for k in ("groups", "pairs", "K", "E", "m", "L"))
        rows = Gn * (K + 1) + 4 * P
        n = 2 * E * m + L * m + 1
        return dict(bytes=rows * 4 * E + Gn * (12 * K + 12) + P * 24 + 7 * 4 * n,
                    flops=2 * E * m * (2 * rows + Gn))
    T, nb = case["rounds"], case["count"]
    # one evaluation of the gain and one of the cost: the log is read once
    return dict(bytes=T * (nb * 8 + 16), flops=T * nb * 60)


def tolerance(case):
    kind = case["kind"]
    if kind == "round":
        # Real outputs are fp32 sums of a row; whole ones follow from them, and
        # a tie closer than their rounding may move one sequence of a batch.
        # Against 64 bits: 5e-8, the largest probability 4e-7.
        t = {"rel": 1e-5, "max": 1e-4}
        if case["batch"] >= 8:
            t["differ"] = min(0.1, 1.2 / case["batch"])
        return t
    if kind == "verify":
        return "exact"
    if kind == "train":
        # against 64 bits: the gradient 3e-7, the rest 3e-8
        return {"rel": 2e-6, "max": 1e-4}
    # against 64 bits: 4e-8, but the optimum of a noisy log is flat
    return {"rel": 2e-6}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _exact_rows(logits, K):
    """Per row: top-K ids (value descending, id ascending), log q, lse, largest
    probability, entropy."""
    B, L, V = logits.shape
    dev = logits.device
    ids = torch.empty(B, L, K, dtype=torch.int64, device=dev)
    logq, lse, mp, ent = (torch.empty(*s, dtype=torch.float64, device=dev)
                          for s in ((B, L, K), (B, L), (B, L), (B, L)))
    for b in range(B):
        x = logits[b].double()
        lse[b] = torch.logsumexp(x, -1)
        lp = x - lse[b][:, None]
        ent[b] = -(lp.exp() * lp).sum(-1)
        mp[b] = lp.max(-1).values.exp()
        h = logits[b].view(torch.int16).long() & 0xFFFF
        key = torch.where(h >= 0x8000, 0xFFFF - h, h + 0x8000)
        key = (key << 32) - torch.arange(V, device=dev)
        ids[b] = torch.topk(key, K, dim=-1).indices
        logq[b] = lp.gather(-1, ids[b])
    return ids, logq, lse, mp, ent


def _exact_tree(edge, cand, n_want, N):
    """Path scores, canonical order, of the n_want best prefixes of one sequence
    whose edge scores are all at most 0: edge [L, K, K] (row 0 at depth 1)."""
    L, K, _ = edge.shape
    levels = []                                  # (score, candidate slot, parent entry)
    score, slot, par = edge[0, 0], np.arange(K), np.full(K, -1)
    allsc = score.copy()
    levels.append((score, slot, par))
    for l in range(1, L):
        thr = -np.inf if allsc.size < n_want else np.partition(allsc, -n_want)[-n_want]
        live = np.flatnonzero(score >= thr)
        if live.size == 0:
            break
        s = score[live][:, None] + edge[l][slot[live]]
        keep = s >= thr
        rr, cc = np.nonzero(keep)
        score, slot, par = s[rr, cc], cc, live[rr]
        levels.append((score, slot, par))
        allsc = np.concatenate([allsc, score])
        if score.size == 0:
            break
    n = min(n_want, allsc.size)
    thr = np.partition(allsc, -n)[-n]
    out = np.zeros(N)
    at, rank = 0, None
    for l, (score, slot, par) in enumerate(levels):
        live = np.flatnonzero(score >= thr)
        up = np.zeros(live.size) if rank is None else rank[par[live]]
        order = np.lexsort((cand[l][slot[live]], up))
        rank = np.full(score.size, -1)
        rank[live[order]] = np.arange(live.size)
        take = score[live[order]][:max(0, N - at)]
        out[at:at + take.size] = take
        at += take.size
    return out


def _exact_round(case, seed):
    d = _round_inputs(case, seed)
    B, L, K, N, m = (case[k] for k in ("batch", "L", "K", "N", "m"))
    ids, logq, lse, mp, ent = _exact_rows(d["logits"], K)
    D = torch.float64
    emb, u = d["emb"].double(), d["u"]
    P, C = emb @ d["g_parent"].double(), emb @ d["g_child"].double()
    u = torch.zeros(L, m, dtype=D, device=emb.device) if u is None else u.double()
    # the ABI's scale is fp32
    scale, beta = float(np.float32(d["scale"])), d["beta"]
    edge = torch.zeros(B, L, K, K, dtype=D, device=emb.device)
    for l in range(L):
        prev = d["root"].long()[:, None] if l == 0 else ids[:, l - 1]
        f = scale / math.sqrt(m) * ((P[prev] + u[l]) @ (C[ids[:, l]] + u[l]).transpose(1, 2))
        if d["center"]:
            f = f - f.mean(-1, keepdim=True)
        edge[:, l, :f.shape[1]] = logq[:, l][:, None, :] + beta * f
    conf, hist = mp.mean(-1), d["hist"].double()
    adj = None
    if case["hidden"]:
        h = d["hidden"].double()
        adj = torch.nn.functional.cosine_similarity(h[:, :-1], h[:, 1:], dim=-1, eps=0.0)
        feat = adj.mean(-1) + adj[:, -1] - adj[:, 0] if L > 1 else torch.zeros_like(conf)
    else:
        feat = ent.mean(-1)
    if case["budget"]:
        tau = torch.zeros_like(conf)
        budget = np.full(B, case["budget"])
    else:
        q = _saba(case)
        f32 = lambda v: float(np.float32(v))
        phi = [f32(v) for v in q["phi"]]
        tau = (phi[0] + phi[1] * conf + phi[2] * feat + phi[3] * hist).clamp(min=q["tau_min"])
        grid = torch.tensor(q["budgets"], dtype=D, device=emb.device)
        U = (1 - torch.exp(-grid / tau[:, None])) / (
            f32(q["c0"]) + f32(q["c1"]) * grid + f32(q["c2"]) * grid * d["prefix"].double()[:, None])
        budget = np.asarray(q["budgets"])[U.argmax(-1).cpu().numpy()]
    scores = None
    if float(edge.max()) <= 0.0:
        e, c = edge.cpu().numpy(), ids.cpu().numpy()
        scores = np.stack([_exact_tree(e[b], c[b], int(min(budget[b], N)), N)
                           for b in range(B)])
    r = dict(budget=None, n_nodes=None, tokens=None, parents=None, pos_ids=None, mask=None,
             topk_ids=None, topk_logq=logq, row_lse=lse, row_maxprob=mp, row_entropy=ent,
             node_scores=scores, saba_state=torch.stack([conf, feat, hist, tau], 1), acc_len=None,
             acc_nodes=None, bonus=None)
    if case["hidden"]:
        r["adj_cos"] = adj
    return r


def _exact_verify(case, seed):
    d = _verify_inputs(case, seed)
    B, L, N = case["batch"], case["L"], case["N"]
    bit = torch.arange(N, device="cuda")
    seen = (d["mask"][:, :, bit >> 6] >> (bit & 63)) & 1
    on = torch.from_numpy(d["on"]).cuda()
    seen = (seen == 1) & on[:, :, None] & on[:, None, :]
    bias = torch.zeros(B, N, (N + 7) // 8 * 8, dtype=torch.float64, device="cuda")
    bias[:, :, :N] = torch.where(seen, 0.0, -math.inf)
    dst = torch.zeros(case["planes"], B, L, case["width"], dtype=torch.bfloat16, device="cuda")
    for b in range(B):
        at, path = -1, []
        kids = {}
        for k in range(int(d["n"][b])):
            kids.setdefault((int(d["par"][b, k]), int(d["tok"][b, k])), k)
        while len(path) < L:
            k = kids.get((at, int(d["tgt"][b, at + 1])))
            if k is None:
                break
            path.append(k)
            at = k
        if path:
            dst[:, b, :len(path)] = d["src"][:, b, path]
    return dict(bias=bias, acc_len=None, acc_nodes=None, bonus=None, dst=dst)


def _exact_train(case, seed):
    d = _train_inputs(case, seed)
    E, m, L, K = (case[k] for k in ("E", "m", "L", "K"))
    h = _hyper(K)
    D = torch.float64
    th = d["theta"].double().requires_grad_(True)
    n = E * m
    gp, gc, u, s = (th[:n].view(E, m), th[n:2 * n].view(E, m),
                    th[2 * n:2 * n + L * m].view(L, m), th[-1])
    emb, b = d["emb"], d["batch"]

    def f(p, c, dep):
        ud = u[dep.long() - 1]
        x = emb[p.long()].double() @ gp + ud
        y = emb[c.long()].double() @ gc + (ud if c.dim() == 1 else ud[:, None, :])
        dot = (x * y).sum(-1) if c.dim() == 1 else (x[:, None, :] * y).sum(-1)
        return s * dot / math.sqrt(m)

    fg = f(b["parent"], b["child"], b["depth"])
    z = torch.log_softmax(b["z"].double(), -1)
    kl = (z.exp() * (z - torch.log_softmax(b["logq"].double() + fg, -1))).sum(-1).mean()
    y = (b["child"] == b["target"][:, None]).to(D)
    ls = torch.nn.functional.logsigmoid
    bce = -(h["w1"] * y * ls(fg) + (1 - y) * ls(-fg)).mean()
    q = b["pairs"]
    pair = torch.nn.functional.softplus(
        h["gamma"] - f(q[:, 0], q[:, 1], q[:, 2]) + f(q[:, 3], q[:, 4], q[:, 5])).mean()
    loss = h["kl"] * kl + h["pair"] * pair + h["bce"] * bce
    (grad,) = torch.autograd.grad(loss, th)
    b1, b2 = h["beta1"], h["beta2"]
    mm = b1 * d["adam_m"].double() + (1 - b1) * grad
    vv = b2 * d["adam_v"].double() + (1 - b2) * grad * grad
    t = TRAIN_STEP
    step = mm / (1 - b1 ** t) / ((vv / (1 - b2 ** t)).sqrt() + h["eps"])
    new = th.detach() * (1 - h["lr"] * h["wd"]) - h["lr"] * step
    return dict(theta=new, adam_m=mm, adam_v=vv,
                loss=torch.stack([loss, kl, pair, bce]).detach(), grad=grad)


def _hyper(K):
    """TdesHyper's defaults as the ABI's fp32 values."""
    f32 = lambda v: float(np.float32(v))
    return dict(kl=1.0, pair=1.0, bce=0.25, gamma=1.0, w1=float(K - 1), lr=f32(2e-3),
                wd=f32(1e-4), beta1=f32(0.9), beta2=f32(0.999), eps=f32(1e-8))


def _exact_fit(case, seed):
    d = _fit_inputs(case, seed)
    D = torch.float64
    B = torch.tensor(d["grid"], dtype=D, device="cuda")
    lat, acc, pre = d["latency"].double(), d["accepted"].double(), d["prefix"].double()
    one = torch.ones_like(lat)
    X = torch.stack([one, one * B, B * pre[:, None]], -1).view(-1, 3)
    size = X.norm(dim=0)
    Q, R = torch.linalg.qr(X / size)
    c = torch.linalg.solve_triangular(R, (Q.T @ lat.reshape(-1, 1)), upper=True).squeeze(1) / size
    cost_sse = ((X @ c - lat.reshape(-1)) ** 2).sum()
    S = torch.cat([torch.ones(lat.shape[0], 1, dtype=D, device="cuda"), d["state"].double()], 1)

    def parts(phi):
        lin = S @ phi
        tau = lin.clamp(min=FIT_TAU_MIN)
        e = torch.exp(-B / tau[:, None])
        Gn = 1 - e
        A = (acc * Gn).sum(1) / (Gn * Gn).sum(1)
        r = A[:, None] * Gn - acc
        w = -A[:, None] * e * B / (tau * tau)[:, None] * (lin > FIT_TAU_MIN)[:, None]
        J = w[:, :, None] * S[:, None, :]
        J = J.reshape(-1, 4)
        return float((r * r).sum()), (J.T @ J).cpu().numpy(), (J.T @ r.reshape(-1)).cpu().numpy()

    phi = np.asarray(FIT_START, np.float64)
    at = lambda p: parts(torch.tensor(p, dtype=D, device="cuda"))
    F, H, gr = at(phi)
    lam = 1e-3
    for _ in range(200):
        step = np.linalg.solve(H + lam * np.diag(np.diag(H)), -gr)
        F2, H2, g2 = at(phi + step)
        if F2 < F:
            done = (F - F2) <= 1e-16 * F
            phi, F, H, gr, lam = phi + step, F2, H2, g2, max(lam / 10, 1e-15)
            if done:
                break
        else:
            lam *= 10
            if lam > 1e14:
                break
    return dict(phi=phi, c=c.cpu().numpy(), sse=np.array([F, float(cost_sse)]))


def exact(case, seed):
    kind = case["kind"]
    return {"round": _exact_round, "verify": _exact_verify, "train": _exact_train,
            "fit": _exact_fit}[kind](case, seed)
