#!/usr/bin/env python3
"""Benchmark of the verify step (forward -> rejection sampling -> KV commit) on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME] [--no-cpu-baseline] [--no-graph]

One "step" is one pass of the whole hot path over one synthetic batch that is resident in HBM
before timing starts.  The K timed steps are recorded once into a HIP graph and its replay is timed
(--no-graph: one host launch per kernel; workloads with a draft model default to that).  Prints ONE JSON line: accepted tokens/s (whole job = this one GPU),
ms/step, the roofline object of the dominant kernel (HIP-event timing of every kernel class over
a second, instrumented run of the same K steps) and the CPU oracle timed on a bounded sample.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X published HBM3E peak
MFMA_BF16_PEAK_TFLOPS = 2500.0 # MI355X published dense bf16 MFMA peak
DEFAULT_WORKLOAD = "llama8b_b32_ctx1k-8k_k3"


def run_steps(wl, sv, torch, n_steps, accept_out, step0, marks=None):
    """n_steps verify steps on the current stream; accept lengths of step i land in accept_out[i].
    A workload with a draft model runs its draft loop first and rolls the draft's cache back afterwards;
    marks (a list) then receives (start, after-draft, end) event triples of every step."""
    sess = wl.sess
    B, k, V = wl.B, wl.k, wl.cfg["vocab"]
    buf = sess.step_buffers(B, k)
    pair = hasattr(wl, "loop")
    draft = wl.loop.drafts if pair else wl.tokens[:, 1:].contiguous()
    T = wl.wl["temperature"]
    ws = buf["workspace"]
    off = (-ws.data_ptr()) % 256
    ws = ws[off:off + ws.numel() - 256]
    for i in range(n_steps):
        wl.restore()                                             # same cache state every step
        if pair:
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)] if marks is not None else None
            if ev:
                ev[0].record()
            wl.loop.run(wl.seq_ids, wl.pending, wl.q, T, wl.seed, step0 + i, pending_hidden=wl.pending_hidden)
            wl.tokens[:, 1:] = draft                             # drafted tokens into the verify input rows
            if ev:
                ev[1].record()
        if pair and wl.tap_layers:                             # ... at several depths (features)
            sv.spec_verify_forward_taps(sess.model, sess.kv, B, k, wl.seq_ids, wl.tokens, buf["logits"], wl.tap_layers, wl.target_hidden, ws)
        elif pair and wl.pending_hidden is not None:          # the draft consumes the target's hidden states: export them
            sv.spec_verify_forward_hidden(sess.model, sess.kv, B, k, wl.seq_ids, wl.tokens, None, buf["logits"], wl.target_hidden, ws)
        else:
            sv.spec_verify_forward(sess.model, sess.kv, B, k, wl.seq_ids, wl.tokens, buf["logits"], ws)
        sv.spec_reject_sample(B, k, V, buf["logits"], wl.q, draft, T, wl.seed, step0 + i, accept_out[i],
                              buf["out_tokens"], None, buf["sample_ws"])
        sv.spec_commit_kv(sess.kv, B, k, wl.seq_ids, accept_out[i], buf["new_ctx_len"], buf["commit_slots"])
        if pair:
            wl.loop.roll_back(wl.seq_ids, buf["new_ctx_len"])
            if ev:
                ev[2].record()
                marks.append(ev)


def replay_ms(sv, torch, record, reps=3):
    """Record what `record()` launches into a HIP graph on a side stream, replay it once untimed, then time `reps` replays."""
    side = torch.cuda.Stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(side):
        sv.spec_graph_capture_begin(side)
        record()
        graph = sv.spec_graph_capture_end(side)
        sv.spec_graph_launch(graph, side)
        side.synchronize()
        e0.record(side)
        for _ in range(reps):
            sv.spec_graph_launch(graph, side)
        e1.record(side)
        side.synchronize()
    torch.cuda.synchronize()
    sv.spec_graph_destroy(graph)
    return e0.elapsed_time(e1) / reps


def hbm_ceiling(sv, torch, nbytes=1 << 30, reps=5):
    """Measured streaming ceiling: the library's plain read and copy kernels over a buffer of known size."""
    src = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    src.zero_()
    dst = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    sink = torch.zeros(4, dtype=torch.uint8, device="cuda")
    out = {}
    for name, fn, moved in (("read", lambda: sv.spec_calib_read(src, nbytes, sink, 512), nbytes),
                            ("copy", lambda: sv.spec_calib_copy(dst, src, nbytes, 1024), 2 * nbytes)):
        fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        out[name + "_GBs"] = round(moved * reps / (e0.elapsed_time(e1) / 1e3) / 1e9, 1)
    out["bytes"] = nbytes
    return out


def cpu_baseline(wl, torch, n_seqs):
    """The CPU oracle, as it stands, on the first n_seqs sequences of the same batch at full depth."""
    import numpy as np

    import synth_inputs as si
    from oracle import commit as oracle_commit
    from oracle import forward as of
    from oracle import sampler as oracle_sampler
    cfg = wl.cfg
    n_seqs = min(n_seqs, wl.B)
    # inputs for the oracle: weights and the sampled sequences' cache, copied to the host (not timed)
    weights = si.make_weights(cfg, seed=wl.seed, device=str(wl.device))
    w_or = si.weights_for_oracle(cfg, weights)
    del weights
    torch.cuda.empty_cache()
    kv_or = [[tuple(t.float().cpu().numpy() for t in wl.logical_kv(l, b)) for b in range(n_seqs)]
             for l in range(cfg["n_layers"])]
    tokens = wl.tokens[:n_seqs].cpu().numpy()
    q = wl.q[:n_seqs].cpu().numpy()
    ctx = wl.ctx_len[:n_seqs]
    book = oracle_commit.KVBook(wl.sess.n_pages, si.PAGE_SIZE)
    for b in range(n_seqs):
        book.assign(b, int(ctx[b]), wl.batch["page_lists"][b])
    t0, c0 = time.perf_counter(), time.process_time()
    logits, _ = of.verify_forward(cfg, w_or, kv_or, tokens, ctx)
    n, _ = oracle_sampler.reject_sample(logits.astype(np.float32), q, tokens[:, 1:], wl.wl["temperature"], wl.seed, 0)
    book.reserve(list(range(n_seqs)), wl.k)
    book.commit(list(range(n_seqs)), n, wl.k)
    dt, cpu = time.perf_counter() - t0, time.process_time() - c0
    try:
        from threadpoolctl import threadpool_info
        pool = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
    except Exception:
        pool = 1
    produced = float((n + 1).sum())
    # threads the oracle actually kept busy: CPU seconds over wall seconds (its matrix products run on the BLAS pool,
    # its attention loops and everything else on one thread)
    busy = max(1, int(round(cpu / dt)))
    return dict(value=produced / dt, unit="accepted tokens/s", cores=busy, kind="oracle",
                sample="%d of %d sequences of the same batch at full depth (%d layers, full vocabulary): forward + rejection "
                       "sampling + commit took %.1f s of wall time and %.1f s of CPU time (BLAS pool of %d threads, the rest "
                       "single-threaded; fp64 conversion of the weights per layer included).  Sequences are independent, so "
                       "the rate stands for the whole batch, which would take about %.0f s"
                       % (n_seqs, wl.B, cfg["n_layers"], dt, cpu, pool, dt * wl.B / n_seqs),
                seconds=dt, blas_threads=int(pool)), logits


def run_continuous(args, wl, sv, torch):
    """Continuous rollout workload: `slots` batch slots over B sequences (the rest wait, prompts cached), long-tailed
    response lengths, n-gram drafter; timed from the first step until every sequence has finished."""
    import numpy as np

    import synth_inputs as si
    from paper_2604_26779_amd.draft import ContinuousRollout
    from paper_2604_26779_amd.workloads import algorithmic_bytes
    n_seqs, slots, k = wl.B, wl.wl["slots"], wl.k
    target = si.response_lengths(wl.wl, wl.seed)
    max_steps = int(target.sum())                               # one token per live slot and step at the very least
    g = torch.Generator(device="cuda")
    g.manual_seed(int(wl.seed) + 9)
    cap = int(wl.ctx_len.max()) + 1 + int(target.max()) + k + 1
    hist0 = torch.randint(0, 12, (n_seqs, cap), generator=g, device="cuda", dtype=torch.int32)
    hist_len0 = torch.from_numpy((wl.ctx_len + 1).astype("int32")).cuda()
    first = hist0[torch.arange(n_seqs, device="cuda"), (hist_len0 - 1).long()].contiguous()
    chunk = 16
    results = {}
    # three passes over the same rollout: a warm-up, a timed one with all slots riding along to the end, and a timed one
    # that moves the live slots to the front and shrinks the batch (in steps of 8 slots) whenever the host looks
    for rep, mode in enumerate(("warm-up", "compacted", "fixed batch")):
        wl.restore()
        hist, hist_len = hist0.clone(), hist_len0.clone()
        roll = ContinuousRollout(wl.sess, slots, k, torch.arange(slots, dtype=torch.int32), torch.from_numpy(target),
                                 torch.arange(slots, n_seqs, dtype=torch.int32), first)
        roll.tokens[:, 0] = first[:slots]
        live = torch.zeros(max_steps + chunk, dtype=torch.int32, device="cuda")
        if mode == "fixed batch":                               # the instrumented pass (events around every kernel class)
            sv.spec_profile_begin((max_steps + chunk) * 420 + 64)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        steps, sizes = 0, []
        while steps < max_steps:                                # the host looks at the live count every `chunk` steps
            sizes.append(roll.B_cur)
            roll.run(hist, hist_len, chunk, wl.wl["temperature"], wl.seed, 9000 + steps, live[steps:steps + chunk])
            steps += chunk
            n_live = roll.compact(granule=8) if mode == "compacted" else int(live[steps - 1].item())
            if n_live == 0:
                break
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        live_h = live[:steps].cpu().numpy()
        used = int(np.argmax(live_h == 0)) + 1 if (live_h == 0).any() else steps
        results[mode] = dict(dt=dt, steps=steps, used=used, live=live_h, produced=int(roll.produced.item()), sizes=sizes)
    prof = sv.spec_profile_end()
    r, fixed = results["compacted"], results["fixed batch"]
    ms_per_step = 1e3 * r["dt"] / r["steps"]
    gemm_ms = sum(prof[n][0] for n in ("gemm_qkv", "gemm_o", "gemm_gu", "gemm_down", "gemm_head")) / fixed["steps"]
    gemm_launches = sum(prof[n][1] for n in ("gemm_qkv", "gemm_o", "gemm_gu", "gemm_down", "gemm_head")) / fixed["steps"]
    alg = algorithmic_bytes(wl.cfg, wl.ctx_len[:slots], slots, k)
    gbs = alg["gemm"] / (gemm_ms / 1e3) / 1e9
    occupancy = float(r["live"][:r["used"]].mean()) / slots
    out = {
        "metric": "accepted tokens/sec/GPU, 8B-shaped verify step k=3; % of HBM/MFMA roofline",
        "value": round(r["produced"] / r["dt"], 1), "unit": "accepted tokens/s", "n_gpus": 1, "steps": r["steps"], "warmup": 0,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": wl.cfg["dtype"], "data": "synthetic",
        "config": {"workload": args.workload, "slots": slots, "sequences": n_seqs, "k": k, "ctx_tokens": int(wl.ctx_len.sum()),
                   "model": wl.wl["model"], "page_size": 16, "pages": "shuffled", "drafter": "n-gram 1..3"},
        "continuous_rollout": {
            "response_tokens": r["produced"], "response_len_min_median_max": [int(target.min()), int(np.median(target)), int(target.max())],
            "steps_until_drained": r["used"], "mean_live_slot_fraction": round(occupancy, 3),
            "steps_with_at_most_a_quarter_live": int((r["live"][:r["used"]] <= slots // 4).sum()),
            "batch_sizes_per_%d_steps" % chunk: r["sizes"],
            "fixed_batch_under_event_profiling": {"tokens_per_s": round(fixed["produced"] / fixed["dt"], 1),
                                                  "ms_per_step": round(1e3 * fixed["dt"] / fixed["steps"], 4)},
            "tokens_per_s_if_all_slots_stayed_live": round(slots * 1e3 / (1e3 * fixed["dt"] / fixed["steps"]), 1),
            "host_syncs": "one every %d steps (live-slot count, batch resize)" % chunk},
        "roofline": dict(kernel="gemm_bf16_kernel", bound="hbm", achieved=round(gbs, 1), peak=HBM_PEAK_GBS, unit="GB/s",
                         frac=round(gbs / HBM_PEAK_GBS, 4), avg_launch_us=round(1e3 * gemm_ms / max(gemm_launches, 1), 2),
                         bytes_per_launch=int(alg["gemm"] / max(gemm_launches, 1)), traffic=None),
        "ms_per_step_by_class": {n: round(ms / fixed["steps"], 4) for n, (ms, cnt) in prof.items() if ms > 0},
    }
    print(json.dumps(out))


def run_continuous_pair(args, wl, sv, torch):
    """The continuous rollout with the draft model as drafter: `slots` batch slots over B sequences, long-tailed response
    lengths; timed from the first step until every sequence has finished (fixed batch: idle slots ride along)."""
    import numpy as np

    import synth_inputs as si
    from paper_2604_26779_amd.draft import ContinuousPairRollout
    n_seqs, slots, k = wl.B, wl.wl["slots"], wl.k
    target = si.response_lengths(wl.wl, wl.seed)
    max_steps = int(target.sum())
    g = torch.Generator(device="cuda")
    g.manual_seed(int(wl.seed) + 9)
    prev = torch.randint(0, wl.cfg["vocab"], (n_seqs,), generator=g, device="cuda", dtype=torch.int32)
    first = torch.from_numpy(wl.batch["tokens0"].astype("int32")).cuda()
    chunk = 16
    results = {}
    for mode in ("warm-up", "timed"):
        wl.restore()
        roll = ContinuousPairRollout(wl.sess, wl.dsess, slots, k, torch.arange(slots, dtype=torch.int32), torch.from_numpy(target),
                                     torch.arange(slots, n_seqs, dtype=torch.int32), prev, first)
        live = torch.zeros(max_steps + chunk, dtype=torch.int32, device="cuda")
        acc = torch.zeros((max_steps + chunk, slots), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        steps = 0
        while steps < max_steps:                                # the host looks at the live count every `chunk` steps
            roll.run(chunk, wl.wl["temperature"], wl.seed, 9000 + steps, live[steps:steps + chunk], acc[steps:steps + chunk])
            steps += chunk
            if int(live[steps - 1].item()) == 0:
                break
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        live_h = live[:steps].cpu().numpy()
        used = int(np.argmax(live_h == 0)) + 1 if (live_h == 0).any() else steps
        results[mode] = dict(dt=dt, steps=steps, used=used, live=live_h, produced=int(roll.produced.item()),
                             alpha=float((acc[:used] + 1).float().mean().item()))
    r = results["timed"]
    out = {
        "metric": "accepted tokens/sec/GPU, 8B-shaped verify step k=3; % of HBM/MFMA roofline",
        "value": round(r["produced"] / r["dt"], 1), "unit": "accepted tokens/s", "n_gpus": 1, "steps": r["steps"], "warmup": 0,
        "ms_per_step": round(1e3 * r["dt"] / r["steps"], 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": wl.cfg["dtype"], "data": "synthetic",
        "config": {"workload": args.workload, "slots": slots, "sequences": n_seqs, "k": k, "ctx_tokens": int(wl.ctx_len.sum()),
                   "model": wl.wl["model"], "draft_model": wl.wl["draft_model"], "page_size": 16, "pages": "shuffled"},
        "continuous_rollout": {
            "response_tokens": r["produced"], "response_len_min_median_max": [int(target.min()), int(np.median(target)), int(target.max())],
            "steps_until_drained": r["used"], "mean_live_slot_fraction": round(float(r["live"][:r["used"]].mean()) / slots, 3),
            "mean_acceptance_length_over_all_slots": round(r["alpha"], 3),
            "host_syncs": "one every %d steps (live-slot count)" % chunk},
        "roofline": None,
    }
    print(json.dumps(out))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default=DEFAULT_WORKLOAD)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seqs", type=int, default=8)
    ap.add_argument("--rollout-steps", type=int, default=8, help="draft+target pair: consecutive steps of the sustained run")
    ap.add_argument("--graph", action="store_true", help="record the K timed steps into a HIP graph and time its replay (the default for the single-model workloads)")
    ap.add_argument("--no-graph", action="store_true", help="one host launch per kernel in the timed region")
    ap.add_argument("--tune", action="append", default=[], help="name=value launch parameter (repeatable)")
    ap.add_argument("--k", type=int, default=None, help="draft length instead of the workload's own (the draft-length sweep of Table 4)")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build measures one GPU (the verify step shards by sequence with no exchange); "
                 "run with --gpus 1")

    import numpy as np
    import torch

    from paper_2604_26779_amd import binding as sv
    import synth_inputs as si
    from paper_2604_26779_amd.workloads import DeviceWorkload, DraftPairWorkload, algorithmic_bytes
    assert torch.cuda.is_available(), "bench.py needs the GPU"
    torch.cuda.set_device(0)
    for item in args.tune:
        name, value = item.split("=")
        sv.spec_tune_set(name, int(value))

    if args.k is not None:
        si.WORKLOADS[args.workload] = dict(si.WORKLOADS[args.workload], k=args.k)
    if "slots" in si.WORKLOADS[args.workload] and "draft_model" in si.WORKLOADS[args.workload]:
        run_continuous_pair(args, DraftPairWorkload(args.workload), sv, torch)
        return
    if "slots" in si.WORKLOADS[args.workload]:
        run_continuous(args, DeviceWorkload(args.workload), sv, torch)
        return
    pair = "draft_model" in si.WORKLOADS[args.workload]
    if pair:
        wl = DraftPairWorkload(args.workload)
    else:
        wl = DeviceWorkload(args.workload)
        wl.make_drafts()
    B, k = wl.B, wl.k
    K, W = args.steps, args.warmup
    accept = torch.zeros((max(K, W), B), dtype=torch.int32, device="cuda")

    run_steps(wl, sv, torch, W, accept, 0)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    args.graph = (args.graph or not pair) and not args.no_graph
    if not args.graph:
        t0 = time.perf_counter()
        ev0.record()
        run_steps(wl, sv, torch, K, accept, 1000)
        ev1.record()
        torch.cuda.synchronize()
    else:
        # the K steps (each with its own random-counter value) are recorded once into a HIP graph on a side stream and
        # replayed: the ~350 launches of a step then cost the GPU's own node-to-node time, not a host launch each
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            sv.spec_graph_capture_begin(side)
            run_steps(wl, sv, torch, K, accept, 1000)
            graph = sv.spec_graph_capture_end(side)
            sv.spec_graph_launch(graph, side)                   # untimed first replay
            side.synchronize()
            t0 = time.perf_counter()
            ev0.record(side)
            sv.spec_graph_launch(graph, side)
            ev1.record(side)
            side.synchronize()
        torch.cuda.synchronize()
        sv.spec_graph_destroy(graph)
    wall = time.perf_counter() - t0
    ms_per_step = ev0.elapsed_time(ev1) / K
    produced = float((accept[:K] + 1).sum().item())          # tokens produced = accepted drafts + 1 per sequence
    accepted_drafts = float(accept[:K].sum().item())
    tokens_per_s = produced / (ms_per_step * K / 1e3)

    # draft / verify split of a pair: events between the two halves of every step, launched kernel by kernel, and the
    # draft loop alone replayed from a HIP graph (K x (cache restore + draft loop) minus K x cache restore)
    marks = [] if pair else None
    draft_loop_graph_ms = None
    if pair:
        run_steps(wl, sv, torch, K, accept, 1000, marks)
        torch.cuda.synchronize()

        def draft_only(with_loop):
            for i in range(K):
                wl.restore()
                if with_loop:
                    wl.loop.run(wl.seq_ids, wl.pending, wl.q, wl.wl["temperature"], wl.seed, 1000 + i, pending_hidden=wl.pending_hidden)
                    wl.tokens[:, 1:] = wl.loop.drafts
        draft_loop_graph_ms = (replay_ms(sv, torch, lambda: draft_only(True)) - replay_ms(sv, torch, lambda: draft_only(False))) / K

    # instrumented run of the same K steps: HIP events around every kernel class
    sv.spec_profile_begin(K * (400 + (200 if pair else 0)) + 64)
    run_steps(wl, sv, torch, K, accept, 1000)
    prof = sv.spec_profile_end()
    per_step = {name: ms / K for name, (ms, cnt) in prof.items()}
    launches = {name: cnt / K for name, (ms, cnt) in prof.items()}
    alg = algorithmic_bytes(wl.cfg, wl.ctx_len, B, k)
    # Every bracket of the instrumented run holds one event record and the idle time around it besides its kernels: the
    # brackets of a step add up to more than the timed step, whose kernels run back to back.  That excess, spread evenly
    # over the brackets, is taken off each class before a launch duration is derived (both figures are reported).
    brackets = sum(launches.values())
    bracket_overhead_ms = max(0.0, sum(per_step.values()) - ms_per_step) / max(brackets, 1.0)
    net = {name: max(per_step[name] - bracket_overhead_ms * launches[name], 0.0) for name in per_step}
    gemm_classes = ("gemm_qkv", "gemm_o", "gemm_gu", "gemm_down", "gemm_head")
    gemm_ms = sum(net[n] for n in gemm_classes)
    gemm_ms_raw = sum(per_step[n] for n in gemm_classes)
    gemm_launches = sum(launches[n] for n in gemm_classes)
    gemm_flops = alg["gemm_flops"]                              # 2 flop per weight an input row meets, per position
    classes = {
        "gemm_bf16_kernel": dict(ms=gemm_ms, raw_ms=gemm_ms_raw, launches=gemm_launches, bytes=alg["gemm"], flops=gemm_flops),
        # (the class also holds the sums of the QKV projection's slices, the rotation and the cache write; its bytes are the cached keys and values alone)
        "attn_partial_kernel": dict(ms=net["attn"], raw_ms=per_step["attn"], launches=launches["attn"], bytes=alg["attn"], flops=0.0),
    }
    dom = max(classes, key=lambda n: classes[n]["ms"])
    # HBM bytes per launch of the dominant kernel by hardware counters: not measured in this run (counters need the
    # profiler); taken from the committed summary of an earlier counter run of the same command, named in traffic_source
    traffic, traffic_source = None, None
    tpath = os.path.join(ROOT, "profiles", "hbm_traffic.json")
    if os.path.exists(tpath):
        entry = json.load(open(tpath)).get(args.workload, {})
        traffic, traffic_source = entry.get(dom), entry.get("_source")

    def roof(c):
        gbs = c["bytes"] / (c["ms"] / 1e3) / 1e9 if c["ms"] > 0 else 0.0
        timing = dict(avg_launch_us=round(1e3 * c["ms"] / max(c["launches"], 1), 2),
                      avg_bracket_us_with_event_overhead=round(1e3 * c["raw_ms"] / max(c["launches"], 1), 2))
        if c["flops"] / c["bytes"] > MFMA_BF16_PEAK_TFLOPS * 1e3 / HBM_PEAK_GBS:      # above the ridge: a contraction
            tf = c["flops"] / (c["ms"] / 1e3) / 1e12 if c["ms"] > 0 else 0.0
            return dict(bound="mfma", achieved=round(tf, 1), peak=MFMA_BF16_PEAK_TFLOPS, unit="TFLOP/s",
                        frac=round(tf / MFMA_BF16_PEAK_TFLOPS, 4), **timing,
                        flops_per_launch=int(c["flops"] / max(c["launches"], 1)), weight_stream_GBs=round(gbs, 1))
        return dict(bound="hbm", achieved=round(gbs, 1), peak=HBM_PEAK_GBS, unit="GB/s", frac=round(gbs / HBM_PEAK_GBS, 4),
                    **timing, bytes_per_launch=int(c["bytes"] / max(c["launches"], 1)))
    roofline = dict(kernel=dom, **roof(classes[dom]), traffic=traffic, traffic_source=traffic_source)
    total_bytes = alg["gemm"] + alg["attn"] + alg["sampler"] + alg["logits_write"]

    out = {
        "metric": "accepted tokens/sec/GPU, 8B-shaped verify step k=3; % of HBM/MFMA roofline",
        "value": round(tokens_per_s, 1), "unit": "accepted tokens/s", "n_gpus": 1, "steps": K, "warmup": W,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": wl.cfg["dtype"], "data": "synthetic",
        "config": {"workload": args.workload, "B": B, "k": k, "ctx_tokens": int(wl.ctx_len.sum()),
                   "model": wl.wl["model"], "page_size": 16, "pages": "shuffled",
                   "kv_cache": "fp8_e4m3 codes, one scale per (layer, kv head)" if wl.cfg.get("kv_dtype") else wl.cfg["dtype"],
                   "matrices": "fp8_e4m3 codes, one scale per output row" if wl.cfg.get("w_dtype") else wl.cfg["dtype"]},
        "verify_steps_per_s": round(1e3 / ms_per_step, 2),
        "mean_acceptance_length": round(produced / (K * B), 3),
        "accepted_draft_tokens_per_s": round(accepted_drafts / (ms_per_step * K / 1e3), 1),
        "step_hbm": {"algorithmic_GB": round(total_bytes / 1e9, 3),
                     "achieved_GBs": round(total_bytes / (ms_per_step / 1e3) / 1e9, 1),
                     "frac_of_peak": round(total_bytes / (ms_per_step / 1e3) / 1e9 / HBM_PEAK_GBS, 4)},
        "roofline": roofline,
        "kernels": {n: roof(c) for n, c in classes.items()},
        "ms_per_step_by_class": {n: round(v, 4) for n, v in per_step.items() if v > 0},
        "event_timing": {"brackets_per_step": round(brackets, 1), "overhead_us_per_bracket": round(1e3 * bracket_overhead_ms, 3),
                         "note": "ms_per_step_by_class are raw event brackets (kernels + one event record + idle time each); their sum "
                                 "minus ms_per_step, spread over the brackets, is taken off before avg_launch_us and the roofline "
                                 "figures are derived"},
        "wall_s_timed_region": round(wall, 3),
        "launch": "HIP graph: the K steps recorded once, replayed" if args.graph else "one host launch per kernel",
        "hbm_ceiling_measured": hbm_ceiling(sv, torch),
    }
    if pair:
        out["draft_verify_split_ms"] = {
            "draft_loop": round(sum(e[0].elapsed_time(e[1]) for e in marks) / K, 4),
            "verify_sample_commit_rollback": round(sum(e[1].elapsed_time(e[2]) for e in marks) / K, 4),
            "draft_loop_replayed_from_a_graph": round(draft_loop_graph_ms, 4),
            "draft_model": wl.wl["draft_model"], "draft_passes": k}
        # sustained rollout: consecutive steps, each feeding the next on the device (no cache restore, no host sync)
        from paper_2604_26779_amd.draft import RolloutLoop
        S = args.rollout_steps
        roll = RolloutLoop(wl.sess, wl.dsess, B, k, tap_layers=wl.tap_layers, token_map=wl.token_map)
        acc_s = torch.zeros((S, B), dtype=torch.int32, device="cuda")
        times = []
        for rep in range(2):                      # first repetition warms up
            wl.restore()
            roll.start(wl.pending[:, 0].contiguous(), wl.pending[:, 1].contiguous(), wl.pending_hidden)
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            roll.run(wl.seq_ids, S, wl.wl["temperature"], wl.seed, 5000, acc_s)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        made = float((acc_s + 1).sum().item())
        out["sustained_rollout"] = {"steps": S, "ms_per_step": round(times[-1] / S, 4),
                                    "accepted_tokens_per_s": round(made / (times[-1] / 1e3), 1),
                                    "mean_acceptance_length": round(made / (S * B), 3)}
        args.no_cpu_baseline = True               # the oracle baseline is reported on the headline workload only
    else:
        # model-free n-gram drafter on the same batch: histories of the contexts' lengths over a small alphabet (so
        # that endings recur), a few consecutive steps of draft -> verify with point-mass drafts -> commit -> history
        # update.  With random weights nothing is accepted; what is reported is what the drafter and its step cost.
        from paper_2604_26779_amd.draft import NgramRollout
        S = args.rollout_steps
        g = torch.Generator(device="cuda")
        g.manual_seed(int(wl.seed) + 9)
        cap = int(wl.ctx_len.max()) + 1 + S * (k + 1)
        hist = torch.randint(0, 12, (B, cap), generator=g, device="cuda", dtype=torch.int32)
        hist_len0 = torch.from_numpy((wl.ctx_len + 1).astype("int32")).cuda()
        roll = NgramRollout(wl.sess, B, k, n_max=3, n_min=1)
        acc_s = torch.zeros((S, B), dtype=torch.int32, device="cuda")
        times = []
        for rep in range(2):                      # first repetition warms up
            wl.restore()
            hist_len = hist_len0.clone()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            roll.run(wl.seq_ids, hist, hist_len, S, wl.wl["temperature"], wl.seed, 7000, acc_s)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(20):
            sv.spec_ngram_draft(B, k, 3, 1, hist, hist_len0, wl.seq_ids, roll.tokens, roll.n_drafted)
        e1.record()
        torch.cuda.synchronize()
        wl.restore()
        out["ngram_drafter"] = {"n": "1..3", "steps": S, "ms_per_step": round(times[-1] / S, 4),
                                "draft_kernel_us": round(1e3 * e0.elapsed_time(e1) / 20, 2),
                                "rows_with_an_occurrence": int((roll.n_drafted > 0).sum().item()),
                                "mean_acceptance_length": round(float((acc_s + 1).sum().item()) / (S * B), 3)}
    if wl.cfg.get("kv_dtype") or wl.cfg.get("w_dtype"):
        args.no_cpu_baseline = True                   # the oracle baseline is reported on the headline workload only
    if not args.no_cpu_baseline:
        base, _ = cpu_baseline(wl, torch, args.cpu_seqs)
        out["cpu_baseline"] = {kk: (round(v, 3) if isinstance(v, float) else v) for kk, v in base.items()}
    print(json.dumps(out))


if __name__ == "__main__":
    main()
