#!/usr/bin/env python3
"""Benchmark of GRAFT's per-round draft-tree construction on one MI355X.

A step is one full round for the whole batch: graft_build_tree (logits pass,
TDES edge scoring, SABA budget, best-first selection, emission and ancestor
mask) followed by graft_accept (greedy acceptance walk), on synthetic drafter
logits already resident in HBM.  The default workload is the batch-64 one
(B=64, L=16, V=128256, K=16, SABA budgets 32..512): the metric's
configuration.  Logit buffers are rotated so that the 256 MB Infinity Cache
cannot serve a round's reads from the previous round.

Prints one JSON line: rounds/s and us/round of K rounds timed back to back;
the logits pass against the HBM roofline, its duration from HIP events
recorded around every stage while the same K rounds run a second time (each
event adds the same few microseconds of stream time: that cost, measured as
the difference between the two passes per event, is subtracted from every
stage, and the events stay out of the headline figure), beside the duration
the committed rocprofv3 summary of the same command reports; the CPU oracle
timed on bounded samples on this host (one thread, and every core of the
process's share over sequences); and, after the headline, the batch-128
workload's 50 rounds chained through the device history ring ("config4").
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
METRIC = "draft-tree rounds/sec and µs/round at B=64; logits-pass HBM GB/s vs peak"


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def source_digest() -> str:
    p = os.path.join(ROOT, "paper_2608_20375_amd", "csrc", "k_logits.hip")
    return hashlib.sha256(open(p, "rb").read()).hexdigest()[:16]


def stored_traffic(workload: int):
    """HBM bytes per logits-pass launch from the committed rocprofv3 PMC
    summary (FETCH_SIZE + WRITE_SIZE, calibrated on a plain copy), valid only
    for the kernel source it was measured on."""
    p = os.path.join(ROOT, "profiles", "logits_pass_w%d_traffic.txt" % workload)
    if not os.path.exists(p):
        return None
    kv = {}
    for line in open(p):
        if ":" in line and not line.startswith(" "):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("k_logits_sha256_16") != source_digest():
        return None
    try:
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def stored_valu(workload: int):
    """VALU issue of the logits pass from the committed rocprofv3 SQ counter
    summary: (fraction of the kernel's span a SIMD issues VALU, that time in
    us), valid only for the kernel source it was measured on."""
    p = os.path.join(ROOT, "profiles", "logits_pass_valu_counters.txt")
    if not os.path.exists(p):
        return None
    kv = {}
    for line in open(p):
        if ":" in line and not line.startswith(" "):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("k_logits_sha256_16") != source_digest():
        return None
    try:
        return (float(kv["valu_busy_frac_w%d" % workload]),
                float(kv["valu_us_per_simd_w%d" % workload]))
    except (KeyError, ValueError):
        return None


def cpu_baseline(w, inp, sc, sp, seconds: float, threads: int = 1):
    """The oracle (plain C, fp64) on this host: whole sequences of the timed
    round (row statistics, top-K, edge scores, budget, selection, emission,
    acceptance walk) until `seconds` have passed, over `threads` threads (one
    sequence per task; the oracle's calls release the GIL).  Scaled to whole
    rounds."""
    import oracle
    import synthetic as S
    from concurrent.futures import ThreadPoolExecutor
    P = oracle.make_params(w.L, w.K, w.n_max, w.V, sc, sp)
    fb = inp.get("fixed_budget")
    td = inp.get("target_depth")

    def one(b):
        r = oracle.build_sequence(P, inp["logits"][b], inp["root_token"][b], inp["base_pos"][b],
                                  inp["prefix_len"][b], 0 if fb is None else fb[b],
                                  float(inp["hist"][b]))
        if td is not None:
            oracle.accept(r["n_nodes"], r["tokens"], r["parents"], w.L, target_depth=td[b])
        else:
            # per-node targets from the synthetic target model's CPU twin, as
            # the GPU round draws them on the device
            n = r["n_nodes"]
            par, tok = r["parents"][:n], r["tokens"][:n]
            ptok = np.where(par < 0, inp["root_token"][b], r["tokens"][np.maximum(par, 0)])
            tn = S.node_targets(w.seed, b, r["depth"][:n], ptok, tok, r["topk_ids"], w.V, w.L, w.K)
            troot = S.node_targets(w.seed, b, [0], [-1], [inp["root_token"][b]], r["topk_ids"],
                                   w.V, w.L, w.K)[0]
            oracle.accept(n, r["tokens"], r["parents"], w.L, int(troot),
                          target_node=np.concatenate([tn, -np.ones(w.n_max - n, np.int32)]))
        return 1

    done = 0
    t0 = time.perf_counter()
    with ThreadPoolExecutor(threads) as ex:
        while True:
            n = min(threads, w.batch) if threads > 1 else 1
            done += sum(ex.map(one, [(done + i) % w.batch for i in range(n)]))
            if time.perf_counter() - t0 >= seconds and done >= threads:
                break
    el = time.perf_counter() - t0
    rounds_per_s = (done / w.batch) / el
    return {"value": rounds_per_s, "unit": "rounds/s", "cores": threads, "kind": "oracle",
            "sample": "%d sequences (%.2f rounds) of the timed round (%d rows x %d bf16 logits "
                      "each; row statistics, top-K, edges, budget, selection, emission, "
                      "acceptance), %d thread%s, fp64, scaled to whole rounds" % (
                          done, done / w.batch, w.L, w.V, threads, "s" if threads > 1 else ""),
            "seconds": el}


def host_threads() -> int:
    """Cores this process may run on, at most 16 (the host share of one GPU)."""
    try:
        n = len(os.sched_getaffinity(0))
    except AttributeError:  # pragma: no cover
        n = os.cpu_count() or 1
    return max(1, min(16, n))


def time_verifier(ctx, w, tb, acc_len, acc_nodes, steps, torch, dev):
    """Per-call time of the verifier-side consumers on the last round's tree
    and acceptance: the bf16 additive bias of the draft block (written once
    per call: batch * N_max^2 * 2 bytes, plus the mask read) and the commit of
    the accepted rows of a key/value cache of 72 planes (36 layers x key and
    value) of 2 KiB rows (8 heads x 128 dims, bf16): 2 * 72 * sum(acc_len) *
    2 KiB bytes read and written."""
    planes, row = 72, 2048
    kv = torch.empty(planes, w.batch, w.n_max, row, dtype=torch.uint8, device=dev)
    bias = torch.empty(w.batch, w.n_max, w.n_max, dtype=torch.bfloat16, device=dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(3):
        ctx.mask_to_bias(tb.n_nodes, tb.mask, bias=bias)
        ctx.commit_accepted(acc_len, acc_nodes, kv)
    torch.cuda.synchronize()

    def timed(call):
        # a sleep kernel ahead of the batch lets the host enqueue every call
        # before the GPU reaches them: the events then time GPU work only
        torch.cuda._sleep(100_000_000)
        e0.record()
        for _ in range(steps):
            call()
        e1.record()
        torch.cuda.synchronize()
        return 1e3 * e0.elapsed_time(e1) / steps

    bias_us = timed(lambda: ctx.mask_to_bias(tb.n_nodes, tb.mask, bias=bias))
    commit_us = timed(lambda: ctx.commit_accepted(acc_len, acc_nodes, kv))
    words = (w.n_max + 63) // 64
    bias_bytes = w.batch * w.n_max * (w.n_max * 2 + words * 8)
    moved = int(acc_len.sum().item())
    commit_bytes = 2 * planes * moved * row
    return {"mask_to_bias_us": bias_us, "bias_bytes": bias_bytes,
            "bias_gbs": bias_bytes / bias_us / 1e3,
            "commit_us": commit_us, "commit_bytes": commit_bytes,
            "commit_gbs": commit_bytes / commit_us / 1e3, "accepted_rows": moved,
            "kv": "%d planes x batch %d x %d rows x %d bytes" % (planes, w.batch, w.n_max, row)}


MFMA_F32_PEAK_TFLOPS = 157.3


def time_training(w, steps, torch, dev, G=4096, P=4096, cpu=True):
    """One TDES training step per call (objectives of eq. tdes-training, their
    gradient and AdamW) on a batch of synthetic target-model traces shaped like
    the workload (its vocabulary, L, K and scorer: E = emb_dim, m = rank): G
    groups of K children and P pairs.  GPU time per step from events around
    `steps` calls queued behind a sleep kernel; algorithmic work per step:
      flops = 2 E m (2 (G (K + 1) + 4 P) + G)   (projection of every parent,
              child and pair row, its weight-gradient contraction, and the
              parent-side matrix-vector product of each group),
      bytes = 4 E (G (K + 1) + 4 P) gathered embedding rows + the traces.
    The oracle's CPU time for the same step is reported beside it."""
    import synthetic as S
    import paper_2608_20375_amd as GR
    sc = S.gen_scorer(w, "paper")
    tr = S.gen_traces(w, G, P)
    E, m, L, K = w.emb_dim, w.rank, w.L, w.K
    theta0 = np.concatenate([sc["g_parent"].ravel(), sc["g_child"].ravel(),
                             sc["depth_emb"].ravel(), [np.float32(sc["scale"])]]).astype(np.float32)
    Tt = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    batch = {k: Tt(v) for k, v in tr.items()}
    emb = Tt(sc["emb"])
    tt = GR.TdesTrainer(w.V, E, m, L, K, G, P)
    theta, m1, m2 = Tt(theta0), torch.zeros(theta0.size, device=dev), torch.zeros(theta0.size, device=dev)
    loss = torch.zeros(4, dtype=torch.float64, device=dev)
    hyper = GR.TdesHyper(w1=float(K - 1))
    for i in range(3):
        tt.step(emb, batch, theta, m1, m2, i + 1, hyper, loss=loss)
    torch.cuda.synchronize()
    first_loss = loss.cpu().numpy().tolist()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(100_000_000)
    e0.record()
    for i in range(steps):
        tt.step(emb, batch, theta, m1, m2, i + 4, hyper)
    e1.record()
    torch.cuda.synchronize()
    if tt.device_status() != 0:
        raise RuntimeError("training step reported invalid ids")
    us = 1e3 * e0.elapsed_time(e1) / steps
    rows = G * (K + 1) + 4 * P
    flops = 2 * E * m * (2 * rows + G)
    nbytes = 4 * E * rows + G * (12 + 12 * K) + 24 * P
    out = {"step_us": us, "steps_per_s": 1e6 / us, "groups": G, "pairs": P,
           "edges_per_s": (G * K + 2 * P) * 1e6 / us,
           "flops_per_step": flops, "tflops": flops / us / 1e6,
           "mfma_f32_frac": flops / us / 1e6 / MFMA_F32_PEAK_TFLOPS,
           "bytes_per_step": nbytes, "gbs": nbytes / us / 1e3,
           "loss_after_3_steps": first_loss,
           "shape": "E=%d m=%d L=%d K=%d V=%d" % (E, m, L, K, w.V)}
    tt.close()
    if cpu:
        from oracle import tdes_train as OT
        h = OT.Hyper(w1=float(K - 1))
        z = np.zeros(theta0.size)
        t0 = time.time()
        OT.train_step(theta0.astype(np.float64), z, z, 1, sc["emb"], tr, h, E, m, L)
        out["cpu_oracle_step_s"] = time.time() - t0
    return out


def time_saba_fit(torch, dev, T=20000, cpu=True):
    """SABA's parameter fit on a synthetic same-prefix replay log of T rounds
    over the 32..512 grid (31 budgets, 5% noise): wall time of the whole fit
    (device sums, host steps, synchronisations), iterations, and the oracle's
    time for the same fit."""
    import synthetic as S
    import paper_2608_20375_amd as GR
    r = S.gen_replay(T, noise=0.05, seed=11)
    Tt = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    args = (r["budgets"], Tt(r["state"]), Tt(r["prefix"]), Tt(r["accepted"]), Tt(r["latency"]),
            r["tau_min"], (10.0, 10.0, 10.0, 10.0))
    GR.saba_fit(*args)
    torch.cuda.synchronize()
    t0 = time.time()
    n = 5
    for _ in range(n):
        out = GR.saba_fit(*args)
    dt = (time.time() - t0) / n
    res = {"rounds": T, "budgets": int(len(r["budgets"])), "fit_ms": 1e3 * dt,
           "iterations": out["iterations"], "phi": out["phi"], "c": out["c"],
           "samples_per_s": T * len(r["budgets"]) * (out["iterations"] + 2) / dt}
    if cpu:
        from oracle import saba_fit as OF
        t0 = time.time()
        OF.fit(r["budgets"], r["state"].astype(np.float64), r["prefix"], r["accepted"],
               r["latency"], r["tau_min"], (10.0, 10.0, 10.0, 10.0))
        res["cpu_oracle_fit_ms"] = 1e3 * (time.time() - t0)
    return res


def run_workload(wid, steps, warmup, rotate, hidden_dim, torch, dev, chain=None):
    """Times `steps` rounds of workload wid back to back on one stream after
    `warmup` untimed ones (graft_build_tree + graft_accept over rotating logit
    buffers), then the same rounds again with the library's stage events, then
    a plain read of the same buffers.  Per-node workloads chain their rounds
    through the device history ring (acceptance pushes acc_len, the next
    round's SABA reads the ring mean)."""
    import synthetic as S
    import paper_2608_20375_amd as G
    w = S.workload(wid)
    t0 = time.time()
    inp = S.gen_round(w, 0)
    sc = S.gen_scorer(w, "literal")
    sp = S.saba_params(w) if w.budget_mode == "saba" else None
    log("workload %d: inputs generated in %.1fs" % (wid, time.time() - t0))

    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = G.Context(w.batch, w.L, w.V, w.K, w.n_max, S.HIST_WINDOW)
    ctx.set_scorer(T(sc["emb"]), T(sc["g_parent"]), T(sc["g_child"]),
                   None if sc["depth_emb"] is None else T(sc["depth_emb"]),
                   sc["scale"], sc["beta"], sc["center"])
    if sp is not None:
        ctx.set_saba(list(sp["grid"]), list(sp["phi"]), sp["tau_min"], sp["c0"], sp["c1"], sp["c2"])

    logit_bytes = w.batch * w.L * w.V * 2
    R = rotate or max(2, math.ceil((1 << 30) / logit_bytes))
    base_logits = T(inp["logits"].view(np.int16))
    bufs = [base_logits] + [base_logits.clone() for _ in range(R - 1)]
    root, base_pos = T(inp["root_token"]), T(inp["base_pos"])
    prefix = T(inp["prefix_len"])
    fixed = T(inp["fixed_budget"]) if "fixed_budget" in inp else None
    node_mode = w.targets == "node"
    hist = None if node_mode else T(inp["hist"])
    if node_mode:
        ctx.set_history(T(inp["hist_ring"]))
    tdepth = T(inp["target_depth"]) if not node_mode else None
    hidden = None
    if hidden_dim:
        hidden = T(S.gen_hidden(w, 0, hidden_dim).view(np.int16))
    tb = G.TreeBuffers(ctx, w.batch)
    acc_len = torch.empty(w.batch, dtype=torch.int32, device=dev)
    acc_nodes = torch.empty(w.batch, w.L, dtype=torch.int32, device=dev)
    bonus = torch.empty(w.batch, dtype=torch.int32, device=dev)
    troot = torch.empty(w.batch, dtype=torch.int32, device=dev)
    tnode = torch.empty(w.batch, w.n_max, dtype=torch.int32, device=dev)
    torch.cuda.synchronize()

    def one_round(i):
        ctx.build_tree(bufs[i % R], root, base_pos, prefix_len=prefix, hist=hist,
                       fixed_budget=fixed, hidden=hidden, out=tb)
        if node_mode:
            ctx.synth_node_targets(w.seed + i, root, tb.n_nodes, tb.tokens, tb.parents,
                                   tb.topk_ids, troot, tnode)
            ctx.accept(tb.n_nodes, tb.tokens, tb.parents, target_root=troot, target_node=tnode,
                       update_history=True, acc_len=acc_len, acc_nodes=acc_nodes, bonus=bonus)
        else:
            ctx.accept(tb.n_nodes, tb.tokens, tb.parents, target_depth=tdepth, acc_len=acc_len,
                       acc_nodes=acc_nodes, bonus=bonus)

    for i in range(warmup):
        one_round(i)
    torch.cuda.synchronize()
    log("workload %d: warmup done (%d rounds)" % (wid, warmup))

    # timed region: `steps` rounds back to back, bracketed by synchronizations
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t_host = time.perf_counter()
    e0.record()
    for i in range(steps):
        one_round(warmup + i)
    enqueue_s = time.perf_counter() - t_host
    e1.record()
    torch.cuda.synchronize()
    host_s = time.perf_counter() - t_host
    ms_per_step = e0.elapsed_time(e1) / steps
    log("workload %d: timed %d rounds: %.4f ms/round (host clock %.4f ms/round; host enqueue "
        "%.4f ms/round)" % (wid, steps, ms_per_step, 1e3 * host_s / steps, 1e3 * enqueue_s / steps))

    # the same rounds again with HIP events recorded around every stage (on the
    # library's stream): per-stage durations, and the logits pass for the roofline
    ctx.profile_begin(steps)
    torch.cuda.synchronize()
    e0.record()
    for i in range(steps):
        one_round(warmup + i)
    e1.record()
    torch.cuda.synchronize()
    ms_events = e0.elapsed_time(e1) / steps
    stage_ms, stage_n = ctx.profile_end()
    stage_avg = [m / n if n else 0.0 for m, n in zip(stage_ms, stage_n)]
    log("workload %d: with stage events: %.4f ms/round; stages ms %s" %
        (wid, ms_events, ["%.4f" % x for x in stage_avg]))

    # Every recorded event adds the same stream time (a marker packet), and a
    # stage's interval holds exactly one of them: take that per-event cost from
    # the two timed passes (with and without events; 4 events per
    # graft_build_tree, 2 per graft_accept) and subtract it from every stage.
    events_per_round = 6
    event_ms = max(0.0, (ms_events - ms_per_step) / events_per_round)
    stage_net = [max(0.0, x - event_ms) for x in stage_avg]
    log("workload %d: per-event stream cost %.4f ms; stages net of it %s" %
        (wid, event_ms, ["%.4f" % x for x in stage_net]))
    k1_s = stage_net[0] * 1e-3
    # stage 0 reads the hidden states too, when they are passed
    pass_bytes = logit_bytes + (w.batch * w.L * hidden_dim * 2 if hidden_dim else 0)
    achieved = pass_bytes / k1_s / 1e9 if k1_s > 0 else 0.0

    # a plain read of the same rotating buffers, back to back: the streaming
    # read rate the logits pass is compared with
    sink = torch.empty(G.READ_STREAM_SINK_WORDS, dtype=torch.int32, device=dev)
    for i in range(3):
        G.read_stream(bufs[i % R], sink)
    torch.cuda.synchronize()
    e0.record()
    for i in range(steps):
        G.read_stream(bufs[i % R], sink)
    e1.record()
    torch.cuda.synchronize()
    read_us = 1e3 * e0.elapsed_time(e1) / steps
    read_gbs = logit_bytes / (read_us * 1e-6) / 1e9
    log("workload %d: plain read of one logits buffer: %.2f us = %.0f GB/s" % (wid, read_us, read_gbs))
    return dict(w=w, inp=inp, sc=sc, sp=sp, ctx=ctx, tb=tb, bufs=bufs, R=R,
                logit_bytes=logit_bytes, pass_bytes=pass_bytes, ms_per_step=ms_per_step, ms_events=ms_events,
                stage_avg=stage_avg, stage_net=stage_net, event_ms=event_ms, achieved=achieved,
                read_us=read_us, read_gbs=read_gbs, acc_len=acc_len, acc_nodes=acc_nodes,
                node_mode=node_mode)


def workload_text(w, R, node_mode):
    return ("B=%d sequences, L=%d, V=%d bf16 logits, K=%d, %s, N_max=%d, scorer d=%d rank %d, "
            "%s targets, %d rotating logit buffers" % (
                w.batch, w.L, w.V, w.K,
                "SABA budgets %d..%d" % (min(w.grid), max(w.grid))
                if w.budget_mode == "saba" else "fixed budget %d" % w.fixed_budget,
                w.n_max, w.emb_dim, w.rank,
                "per-node (device history ring chained round to round)" if node_mode
                else "per-depth", R))


def stored_kernel_us(workload: int):
    """Average duration of the logits pass at this workload from the committed
    rocprofv3 kernel-trace summary of the default bench.py command (which
    times the batch-64 headline and then the batch-128 chained rounds), valid
    only for the kernel source it was measured on."""
    p = os.path.join(ROOT, "profiles", "kernels_w3_kernel_trace.txt")
    if not os.path.exists(p):
        return None
    kv = {}
    for line in open(p):
        if ":" in line and not line.startswith(" "):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("k_logits_sha256_16") != source_digest():
        return None
    try:
        return float(kv["logits_pass_avg_us_w%d" % workload])
    except (KeyError, ValueError):
        return None


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", type=int, default=3)
    ap.add_argument("--rotate", type=int, default=0, help="logit buffers (0: >= 1 GiB total)")
    ap.add_argument("--cpu-seconds", type=float, default=8.0,
                    help="single-thread oracle leg: seconds of sequences to time")
    ap.add_argument("--cpu-seconds-all", type=float, default=3.0,
                    help="all-cores oracle leg (threads over sequences): seconds to time")
    ap.add_argument("--config4-steps", type=int, default=50,
                    help="after the batch-64 headline, time this many chained rounds of the "
                         "batch-128 workload (0: skip)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--hidden-dim", type=int, default=0,
                    help="also pass drafter hidden states of this width (SABA uses their "
                         "degeneration signal); 0: the mean-entropy state of the workload")
    ap.add_argument("--verifier", action="store_true",
                    help="also time the verifier-side consumers after the headline: the bf16 "
                         "attention bias of the draft block and the commit of the accepted "
                         "rows in a key/value cache of 72 planes of 2 KiB rows")
    ap.add_argument("--train", action="store_true",
                    help="also time one TDES training step (4096 groups, 4096 pairs of synthetic "
                         "traces with the workload's vocabulary, L, K and scorer sizes)")
    ap.add_argument("--saba-fit", action="store_true",
                    help="also time SABA's parameter fit on a synthetic replay log (20000 "
                         "rounds x 31 budgets)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain device copy of known size (PMC calibration)")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py runs on one GPU only: the draft-tree path shards by sequence with no "
              "communication, so a multi-GPU figure adds nothing here (got --gpus %d, "
              "WORLD_SIZE %d)" % (args.gpus, world), file=sys.stderr)
        sys.exit(2)

    import torch

    import synthetic as S
    import paper_2608_20375_amd as G

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    run = run_workload(args.workload, args.steps, args.warmup, args.rotate, args.hidden_dim,
                       torch, dev)
    w, ctx, tb = run["w"], run["ctx"], run["tb"]
    bufs, R = run["bufs"], run["R"]
    logit_bytes, pass_bytes = run["logit_bytes"], run["pass_bytes"]
    ms_per_step, ms_events = run["ms_per_step"], run["ms_events"]
    stage_avg, stage_net, event_ms = run["stage_avg"], run["stage_net"], run["event_ms"]
    achieved, read_gbs = run["achieved"], run["read_gbs"]
    acc_len, acc_nodes = run["acc_len"], run["acc_nodes"]
    traffic = stored_traffic(args.workload)
    prof_us = stored_kernel_us(args.workload)
    valu = stored_valu(args.workload)

    if args.copy_calibration:
        n = 256 << 20
        src = torch.empty(n, dtype=torch.uint8, device=dev).fill_(1)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        log("copy calibration: 3 copies of %d bytes" % n)

    verifier = None
    if args.verifier:
        verifier = time_verifier(ctx, w, tb, acc_len, acc_nodes, args.steps, torch, dev)
        log("verifier consumers: %s" % verifier)

    training = None
    if args.train:
        training = time_training(w, args.steps, torch, dev, cpu=not args.no_cpu_baseline)
        log("tdes training step: %s" % training)

    saba_fit = None
    if args.saba_fit:
        saba_fit = time_saba_fit(torch, dev, cpu=not args.no_cpu_baseline)
        log("saba fit: %s" % saba_fit)

    nodes = tb.n_nodes.float().mean().item()
    budgets = tb.budget.float().mean().item()
    cpu = None
    if not args.no_cpu_baseline:
        inp, sc, sp = run["inp"], run["sc"], run["sp"]
        one = cpu_baseline(w, inp, sc, sp, args.cpu_seconds)
        log("cpu baseline, 1 thread: %.4f rounds/s over %.1fs" % (one["value"], one["seconds"]))
        nt = host_threads()
        cpu = cpu_baseline(w, inp, sc, sp, args.cpu_seconds_all, threads=nt)
        log("cpu baseline, %d threads: %.4f rounds/s over %.1fs" % (nt, cpu["value"], cpu["seconds"]))
        cpu.pop("seconds")
        one.pop("seconds")
        cpu["single_thread"] = one

    # the batch-128 workload (L=32, V=151936, K=32), 50 rounds chained through
    # the device history ring on one stream: its own round time and logits-pass
    # roofline (no CPU leg)
    config4 = None
    if args.workload == 3 and args.config4_steps > 0:
        del bufs, run
        ctx.close()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        r4 = run_workload(4, args.config4_steps, 5, 0, 0, torch, dev)
        k1 = r4["stage_net"][0]
        config4 = {
            "workload": workload_text(r4["w"], r4["R"], r4["node_mode"]),
            "rounds": args.config4_steps,
            "us_per_round": 1e3 * r4["ms_per_step"],
            "rounds_per_s": 1e3 / r4["ms_per_step"],
            "mean_nodes": r4["tb"].n_nodes.float().mean().item(),
            "stage_us": {"logits_pass": 1e3 * k1, "edge_scores_and_saba": 1e3 * r4["stage_net"][1],
                         "select_emit_mask": 1e3 * r4["stage_net"][2],
                         "accept": 1e3 * r4["stage_net"][3]},
            "logits_pass": {"achieved": r4["achieved"], "unit": "GB/s",
                            "frac": r4["achieved"] / HBM_PEAK_GBS,
                            "algorithmic_bytes_per_launch": r4["logit_bytes"],
                            "plain_read_gbs": r4["read_gbs"],
                            "profile_kernel_us": stored_kernel_us(4),
                            "valu_busy_frac": (stored_valu(4) or (None,))[0]},
        }
        if config4["logits_pass"]["profile_kernel_us"]:
            config4["logits_pass"]["profile_frac"] = (
                r4["logit_bytes"] / (config4["logits_pass"]["profile_kernel_us"] * 1e-6) / 1e9
                / HBM_PEAK_GBS)
        r4["ctx"].close()
        ctx = None

    result = {
        "metric": METRIC,
        "value": 1e3 / ms_per_step,
        "unit": "rounds/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "us_per_round": 1e3 * ms_per_step,
        "us_per_round_with_stage_events": 1e3 * ms_events,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "fp32",
        "data": "synthetic",
        "config": {
            "workload": workload_text(w, R, w.targets == "node"),
            "global_batch": w.batch,
            "hidden_dim": args.hidden_dim,
            "mean_budget": budgets,
            "mean_nodes": nodes,
            "stage_us": {"logits_pass": 1e3 * stage_net[0], "edge_scores_and_saba": 1e3 * stage_net[1],
                         "select_emit_mask": 1e3 * stage_net[2], "accept": 1e3 * stage_net[3]},
            "stage_us_raw_events": [1e3 * x for x in stage_avg],
            "event_overhead_us": 1e3 * event_ms,
        },
        "roofline": {
            "bound": "hbm",
            "kernel": "logits_pass_kernel",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": traffic,
            "algorithmic_bytes_per_launch": pass_bytes,
            "plain_read_gbs": read_gbs,
            "frac_of_plain_read": achieved / read_gbs if read_gbs > 0 else None,
            "kernel_us": 1e3 * stage_net[0],
            "profile_kernel_us": prof_us,
            "profile_frac": (logit_bytes / (prof_us * 1e-6) / 1e9 / HBM_PEAK_GBS
                             if prof_us else None),
            # the secondary bound: share of the kernel's span a SIMD spends
            # issuing VALU, from the committed SQ counter summary
            "valu_busy_frac": valu[0] if valu else None,
            "valu_us_per_simd": valu[1] if valu else None,
        },
        "cpu_baseline": cpu,
    }
    if config4 is not None:
        result["config4"] = config4
    if verifier is not None:
        result["verifier"] = verifier
    if training is not None:
        result["tdes_training"] = training
    if saba_fit is not None:
        result["saba_fit"] = saba_fit
    print(json.dumps(result), flush=True)
    if ctx is not None:
        ctx.close()


if __name__ == "__main__":
    main()
