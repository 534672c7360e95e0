"""Decode-step benchmark of MLKV decode attention on one MI355X.

A step is one pass of the whole hot path over one batch of synthetic input:
for every layer, the owning layers append the newest token's K/V, then every
query head attends over its (shared) KV head through split-K decode attention
(mlkv_decode_step through the C ABI).  Inputs are resident in HBM before the
timed region starts.

Prints ONE JSON line:
  value = algorithmic decode-attention bytes per step / step time (GB/s),
  plus steps/s, the roofline object of the dominant kernel (split-K
  attention, timed per launch with HIP events on the launch stream) and the
  CPU-oracle baseline on the host cores.

  python bench.py [--steps K] [--warmup W] [--workload NAME] [--no-cold]

A workload with T > 1 new tokens per sequence (prefill_b8_2000) runs the
prefill instead (mlkv_prefill_step: owners store the prompt's rows, every
layer attends causally): value = algorithmic attention TFLOP/s, with the
prefill kernel's roofline against the bf16 matrix-core peak.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published
DEFAULT_WORKLOAD = "mlkv4_b128_ragged"
REF_COPY_BYTES = 256 << 20
SLEEP_CYCLES = 40_000_000  # ~17 ms at 2.4 GHz: longer than the host needs to enqueue 10 steps
MFMA_BF16_PEAK_TFLOPS = 2500.0  # MI355X dense bf16 matrix cores, published
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "attention_kernel_traffic.md")
# The decode kernels and the host planner that picks their launch shapes
# (both decide the bytes a launch moves).
KERNEL_SOURCES = [os.path.join(ROOT, "paper_2406_09297_amd", "csrc", f)
                  for f in ("kernels.hip", "tile.h", "mlkv.cpp")]


def kernel_code_sha256() -> str:
    """SHA-256 over the decode kernels' code and the host planner
    (kernels.hip, tile.h, then mlkv.cpp) with comments removed and whitespace
    collapsed, so that editing a comment does not void a counter record taken
    from the same code."""
    import hashlib
    import re

    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(f) as fh:
            text = fh.read()
        text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
        text = re.sub(r"//[^\n]*", " ", text)
        h.update(re.sub(r"\s+", " ", text).strip().encode())
    return h.hexdigest()


def measured_traffic(workload: str):
    """HBM bytes per timed attention launch (the attention kernel plus, where
    one follows it, the merge kernel) from the committed rocprofv3 counter
    summary, or None if it does not cover this workload or the kernels' code
    changed since the counters were taken."""
    try:
        text = open(TRAFFIC_FILE).read()
        sha = kernel_code_sha256()
    except OSError:
        return None
    fields = {}
    for line in text.splitlines():
        line = line.strip().strip("`")
        if "=" in line and not line.startswith("#"):
            k, v = line.split("=", 1)
            fields[k.strip()] = v.strip()
    if fields.get("kernel_code_sha256") != sha:
        return None
    v = fields.get(f"traffic_bytes_per_launch[{workload}]")
    return int(v) if v else None


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def step_bytes(w, ctx, kv_count, owned_count, out_bytes=4):
    """Algorithmic HBM bytes of one step, by layer: every cached K/V byte of the
    KV heads a layer reads, read once per layer; q read; output written; the
    appended rows read and written in owning layers."""
    L = ctx.astype(np.int64) + 1
    per_layer = []
    for n in range(w.l):
        kv = kv_count[n] * int(L.sum()) * w.D * 2 * 2
        q = w.B * w.h * w.D * 2
        out = w.B * w.h * w.D * out_bytes
        app = owned_count[n] * w.B * w.D * 2 * 2 * 2
        per_layer.append(dict(kv=kv, q=q, out=out, append=app))
    return per_layer


def kv_bytes_once(w, ctx):
    """Bytes of the attended rows of every KV head, each read once per step."""
    return w.n_kv * int((np.asarray(ctx, np.int64) + 1).sum()) * w.D * 2 * 2


def cpu_baseline(w, inp, kv_of, owner_of, bytes_per_step, budget_s=10.0, rotary=(0, 1e4)):
    """The oracle, as it stands, on the host cores: whole decode steps on the
    same host inputs, repeated until the time budget is used (at least once);
    then on one thread for a third of that budget (steps of the first
    sequences only if one whole step would not fit it)."""
    import oracle

    threads = oracle.threads()

    def timed(budget, batch):
        sl = slice(0, batch)
        q = np.ascontiguousarray(inp["q"][:, sl])
        kn, vn, ctx = inp["k_new"][sl], inp["v_new"][sl], inp["ctx"][sl]
        runs, spent, t0 = 0, 0.0, time.perf_counter()
        while runs == 0 or time.perf_counter() - t0 < budget:
            k = np.ascontiguousarray(inp["k_cache"][:, sl])
            v = np.ascontiguousarray(inp["v_cache"][:, sl])
            ts = time.perf_counter()
            if rotary[0]:
                oracle.decode_step_rope(q, k, v, kn, vn, kv_of, owner_of, ctx, rotary[0],
                                        rotary[1])
            else:
                oracle.decode_step(q, k, v, kn, vn, kv_of, owner_of, ctx)
            spent += time.perf_counter() - ts
            runs += 1
        return runs, spent

    runs, spent = timed(budget_s, w.B)
    result = {"value": bytes_per_step * runs / spent / 1e9, "unit": "GB/s", "cores": threads,
              "kind": "oracle", "steps_per_s": runs / spent,
              "sample": f"{runs} whole decode step(s) of the same workload (fp64 oracle, "
                        f"OpenMP over (sequence, head)), {spent:.1f} s"}
    # One thread: whole steps of the first n sequences, n sized to the budget.
    per_seq_s = spent / runs / w.B * threads
    n = max(1, min(w.B, int(budget_s / 3 / max(per_seq_s, 1e-9))))
    oracle.threads(1)
    try:
        r1, s1 = timed(budget_s / 3, n)
    finally:
        oracle.threads(threads)
    frac = float((inp["ctx"][:n].astype(np.int64) + 1).sum()) / float((inp["ctx"].astype(np.int64) + 1).sum())
    result["single_thread"] = {
        "value": bytes_per_step * frac * r1 / s1 / 1e9, "unit": "GB/s", "cores": 1,
        "sample": f"{r1} decode step(s) of the first {n} of {w.B} sequences, {s1:.1f} s"}
    return result


def prefill_flops(w, ctx):
    """Algorithmic flops of one prefill (all layers): every (query row, key
    position) pair the causal mask admits costs 2*D for q.k and 2*D for the
    weighted value sum."""
    pairs = sum(int(c) * w.T + w.T * (w.T + 1) // 2 for c in ctx)  # per query head
    return w.l * w.h * pairs * 4 * w.D


def run_prefill(args, w, emit: bool = True):
    import torch
    import synth
    import paper_2406_09297_amd as mlkv

    dev = "cuda:0"
    log(f"[bench] prefill workload {w.name}: generating inputs")
    inp = synth.prefill_inputs(w, fill=0)
    S = inp["capacity"]
    mp = mlkv.Map.uniform(w.l, w.h, w.m, w.g)
    cache = mlkv.Cache.empty(w.n_kv, w.B, S, w.D, dev)
    log("[bench] uploading")
    cache.load_rows(inp["k_cache"], inp["v_cache"])
    q = mlkv.bf16_tensor(inp["q"], dev)
    kn = mlkv.bf16_tensor(inp["k_new"], dev)
    vn = mlkv.bf16_tensor(inp["v_new"], dev)
    ctx = torch.from_numpy(inp["ctx"]).to(dev)
    out = torch.empty((w.l, w.B, w.T, w.h, w.D), dtype=torch.float32, device=dev)
    stream = torch.cuda.current_stream()
    flops = prefill_flops(w, inp["ctx"])
    tokens = w.B * w.T

    def one_step():
        mlkv.prefill_step(q, kn, vn, cache, mp, ctx, out)

    if args.pmc_pass:  # counter pass: one warm prefill, then two in the timed configuration
        for _ in range(3):
            one_step()
        torch.cuda.synchronize()
        log("[bench] pmc pass done")
        return

    log(f"[bench] warmup {args.warmup}")
    for _ in range(args.warmup):
        one_step()
    torch.cuda.synchronize()
    log(f"[bench] timing {args.steps} prefills")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        one_step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms_step = e0.elapsed_time(e1) / args.steps

    log("[bench] timing prefill kernels (event pairs)")
    mlkv.profile_enable(args.steps * w.l)
    torch.cuda.synchronize()
    done = 0
    while done < args.steps:
        n = min(10, args.steps - done)
        torch.cuda._sleep(SLEEP_CYCLES)
        for _ in range(n):
            one_step()
        torch.cuda.synchronize()
        done += n
    n_launch, tot_ms, min_ms, max_ms = mlkv.profile_read()
    durations = mlkv.profile_durations(n_launch)
    mlkv.profile_disable()
    avg = tot_ms * 1e-3 / n_launch
    p10, p50, p90 = (float(np.percentile(durations, pq)) for pq in (10, 50, 90))
    flops_launch = flops * args.steps / n_launch  # a launch is a layer, or all of them
    achieved = flops_launch / avg / 1e12
    result = {
        "metric": "prefill-attention TFLOP/s (% of bf16 MFMA peak) + prompt tokens/s, "
                  "MLKV Pythia-160M shape",
        "value": round(flops / (ms_step * 1e-3) / 1e12, 2),
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "prompt_tokens_per_s": round(tokens / (ms_step * 1e-3), 0),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) bf16 q/K/V; no weights)",
        "config": {"workload": w.name, "l": w.l, "h": w.h, "m": w.m, "g": w.g, "head_dim": w.D,
                   "batch": w.B, "ctx": w.ctx, "new_tokens": w.T, "capacity": S,
                   "flops_per_step": int(flops)},
        "roofline": {"bound": "mfma", "achieved": round(achieved, 2),
                     "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                     "frac": round(achieved / MFMA_BF16_PEAK_TFLOPS, 4), "traffic": None,
                     "kernel": "prefill_kernel", "avg_launch_us": round(avg * 1e6, 2),
                     "min_launch_us": round(min_ms * 1e3, 2),
                     "max_launch_us": round(max_ms * 1e3, 2),
                     "p10_p50_p90_launch_us": [round(p10 * 1e3, 2), round(p50 * 1e3, 2),
                                               round(p90 * 1e3, 2)],
                     "launches": n_launch, "flops_per_launch": int(flops_launch)},
    }
    if not args.no_cpu_baseline:
        log("[bench] cpu baseline (oracle)")
        import oracle

        kv_of, _ = oracle.map_uniform(w.l, w.h, w.m, w.g)
        # Bounded sample: layer 0 of the first sequence (its owners' rows
        # stored first), repeated for about 10 s.
        k, v = inp["k_cache"][:, :1].copy(), inp["v_cache"][:, :1].copy()
        _, owner_of = oracle.map_uniform(w.l, w.h, w.m, w.g)
        oracle.append_rows(0, k, v, inp["k_new"][:1], inp["v_new"][:1], owner_of, inp["ctx"][:1])
        one = w.__class__(w.name, w.l, w.h, w.m, w.g, w.D, 1, w.ctx, w.ctx_range, w.k_scale,
                          w.seed, w.note, T=w.T)
        sample_flops = prefill_flops(one, inp["ctx"][:1]) / w.l
        threads = int(os.environ.get("OMP_NUM_THREADS", len(os.sched_getaffinity(0))))
        runs, spent = 0, 0.0
        while spent < 10.0 or runs == 0:
            ts = time.perf_counter()
            oracle.prefill_attention(0, inp["q"][0, :1], k, v, kv_of, inp["ctx"][:1])
            spent += time.perf_counter() - ts
            runs += 1
        result["cpu_baseline"] = {
            "value": round(sample_flops * runs / spent / 1e12, 6), "unit": "TFLOP/s",
            "cores": threads, "kind": "oracle",
            "prompt_tokens_per_s": round(w.T * runs / spent / w.l, 1),
            "sample": f"{runs} x layer 0 of one sequence ({w.T} tokens, fp64 oracle, "
                      f"OpenMP over (token, head)), {spent:.1f} s; tokens/s scaled to all "
                      f"{w.l} layers"}
    if emit:
        print(json.dumps(result), flush=True)
    return result


def run_model(args, w, emit: bool = True):
    """Whole-model decode step (mlkv_model_decode_step): tokens/s at batch B."""
    import torch
    import synth
    import paper_2406_09297_amd as mlkv

    dev = "cuda:0"
    log(f"[bench] model workload {w.name}: generating weights and cache")
    mp = mlkv.Map.uniform(w.l, w.h, w.m, w.g)
    owned = [mp.layer_owned(n)[1] for n in range(w.l)]
    weights = synth.model_weights(w.seed, w.l, w.h, w.D, w.d_ff, owned)
    dev_w = [{k: (None if v is None else mlkv.bf16_tensor(v, dev)) for k, v in lw.items()}
             for lw in weights]
    d = w.h * w.D
    model = mlkv.Model(mp, d, w.d_ff, w.D, dev_w, rotary_dims=16)
    inp = synth.step_inputs(w, fill=0)
    S = inp["capacity"]
    cache = mlkv.Cache.empty(w.n_kv, w.B, S, w.D, dev)
    cache.load_rows(inp["k_cache"], inp["v_cache"])
    x0 = synth.bf16_to_f32(synth.normal_bf16(w.seed, 0, (w.B, d)))
    x = torch.from_numpy(x0.copy()).to(dev)
    ctx = torch.from_numpy(inp["ctx"]).to(dev)
    ws = model.workspace(w.B, S, dev)
    max_len = int(inp["ctx"].max()) + 1
    stream = torch.cuda.current_stream()

    def one_step():
        model.decode_step(x, cache, ctx, ws, max_len_hint=max_len)

    log(f"[bench] warmup {args.warmup}")
    for _ in range(args.warmup):
        one_step()
    torch.cuda.synchronize()
    log(f"[bench] timing {args.steps} eager model steps")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        one_step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms_eager = e0.elapsed_time(e1) / args.steps
    ms_step = ms_eager
    if not args.no_graph:
        # The step captured once in a HIP graph and replayed: the ~140
        # dependent launches of a step go to the GPU without host launch
        # gaps (replays equal the eager step bit for bit: GPU test).
        log("[bench] capturing one model step in a HIP graph")
        side = torch.cuda.Stream()
        side.wait_stream(stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            one_step()
        torch.cuda.synchronize()
        for _ in range(max(args.warmup, 1)):
            graph.replay()
        torch.cuda.synchronize()
        log(f"[bench] timing {args.steps} graph replays")
        e0.record(stream)
        for _ in range(args.steps):
            graph.replay()
        e1.record(stream)
        torch.cuda.synchronize()
        ms_step = e0.elapsed_time(e1) / args.steps
    # attention launches of the same steps, timed by the library's event pairs
    mlkv.profile_enable(args.steps * w.l)
    done = 0
    while done < args.steps:
        n = min(10, args.steps - done)
        torch.cuda._sleep(SLEEP_CYCLES)
        for _ in range(n):
            one_step()
        torch.cuda.synchronize()
        done += n
    n_launch, tot_ms, _, _ = mlkv.profile_read()
    mlkv.profile_disable()
    attn_ms_step = tot_ms / args.steps
    weight_bytes = sum(int(v.size) * 2 for lw in weights for v in lw.values() if v is not None)
    L = inp["ctx"].astype(np.int64) + 1
    kv_bytes = sum(mp.layer_kv_count(n) for n in range(w.l)) * int(L.sum()) * w.D * 2 * 2
    step_bytes = weight_bytes + kv_bytes
    achieved = step_bytes / (ms_step * 1e-3) / 1e9
    result = {
        "metric": "whole-model decode tokens/s (MLKV Pythia-160M shape, synthetic weights)",
        "value": round(w.B / (ms_step * 1e-3), 1),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded bf16 weights std 0.02, N(0,1) cache; no trained weights)",
        "config": {"workload": w.name, "l": w.l, "h": w.h, "m": w.m, "g": w.g, "head_dim": w.D,
                   "d_model": d, "d_ff": w.d_ff, "batch": w.B, "ctx": w.ctx, "capacity": S,
                   "weight_bytes": weight_bytes, "kv_bytes_per_step": kv_bytes},
        "launch": "one HIP graph per step" if not args.no_graph else "eager launches",
        "eager_ms_per_step": round(ms_eager, 4),
        "attention_ms_per_step": round(attn_ms_step, 4),
        "attention_share": round(attn_ms_step / ms_step, 3),
        "attention_launches_carry": "the MLP's second product (f W_2 + b_2) on the fused path",
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None,
                     "kernel": "whole step (weights read once + KV rows read once per layer)"},
    }
    if not args.no_cpu_baseline:
        log("[bench] cpu baseline (oracle)")
        import oracle
        import oracle.model as om

        kv_of, owner_of = oracle.map_uniform(w.l, w.h, w.m, w.g)

        kc, vc = om._f64(inp["k_cache"]), om._f64(inp["v_cache"])
        threads = int(os.environ.get("OMP_NUM_THREADS", len(os.sched_getaffinity(0))))
        runs, spent = 0, 0.0
        while spent < 10.0 or runs == 0:
            ts = time.perf_counter()
            om.decode_step_model(x0.astype(np.float64), weights, kv_of, owner_of, kc, vc,
                                 inp["ctx"], w.h, w.D, 16)
            spent += time.perf_counter() - ts
            runs += 1
        result["cpu_baseline"] = {
            "value": round(w.B * runs / spent, 2), "unit": "tokens/s", "cores": threads,
            "kind": "oracle",
            "sample": f"{runs} whole model step(s) of the same workload (float64 numpy oracle), "
                      f"{spent:.1f} s"}
    if emit:
        print(json.dumps(result), flush=True)
    return result


CAPACITY_MARGIN = 4 << 30  # device bytes left free beside the step's buffers


def capacity_setup(w, dev, seed):
    """Allocate the largest batch of a decode step at ctx = w.ctx whose cache
    (capacity w.capacity) and step buffers fit in the free device memory, and
    fill it from a seeded device generator (keys, values, queries and new rows
    N(0,1) in bf16).  Returns (B, cache, q, k_new, v_new, ctx, out)."""
    import torch
    import synth
    import paper_2406_09297_amd as mlkv

    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    S = w.capacity
    B = synth.capacity_batch(w, free - CAPACITY_MARGIN, S)
    while True:  # the allocator may not hand out all of it in these pieces
        try:
            cache = mlkv.Cache.empty(w.n_kv, B, S, w.D, dev)
            q = torch.empty((w.l, B, w.h, w.D), dtype=torch.bfloat16, device=dev)
            out = torch.empty((w.l, B, w.h, w.D), dtype=torch.bfloat16, device=dev)
            kn = torch.empty((B, w.n_kv, w.D), dtype=torch.bfloat16, device=dev)
            vn = torch.empty((B, w.n_kv, w.D), dtype=torch.bfloat16, device=dev)
            break
        except torch.OutOfMemoryError:
            cache = q = out = kn = vn = None
            torch.cuda.empty_cache()
            B = int(B * 0.98)
            log(f"[bench] capacity: allocation failed, retrying at batch {B}")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    for t in (cache.k, cache.v, q, kn, vn):
        t.normal_(generator=gen)
    ctx = torch.full((B,), w.ctx, dtype=torch.int32, device=dev)
    torch.cuda.synchronize()
    return B, cache, q, kn, vn, ctx, out


def run_capacity(args, w):
    """The largest batch a 2048-token cache allows on this GPU (the paper's
    memory experiment: 2000 cached tokens, then decode), and decode steps
    timed at that batch."""
    import torch
    import synth
    import paper_2406_09297_amd as mlkv

    dev = "cuda:0"
    hbm_ref = read_reference(64 << 20)["hbm_2GiB_gbs"]  # before the batch takes the memory
    log(f"[bench] capacity workload {w.name}: sizing and filling the batch")
    B, cache, q, kn, vn, ctx, out = capacity_setup(w, dev, w.seed)
    S = w.capacity
    mp = mlkv.Map.uniform(w.l, w.h, w.m, w.g)
    log(f"[bench] capacity: batch {B}, cache {cache.k.numel() * 4 / 1e9:.1f} GB")
    stream = torch.cuda.current_stream()
    L = w.ctx + 1
    kv_count = [mp.layer_kv_count(n) for n in range(w.l)]
    kv_bytes = sum(kv_count) * B * L * w.D * 2 * 2
    qo_bytes = w.l * B * w.h * w.D * (2 + 2)
    owned = sum(mp.layer_owned(n)[1] for n in range(w.l))
    step_total = kv_bytes + qo_bytes + owned * B * w.D * 2 * 2 * 2

    def one_step():
        mlkv.decode_step(q, kn, vn, cache, mp, ctx, out, max_len_hint=L, ws=None)

    log(f"[bench] warmup {args.warmup}")
    for _ in range(args.warmup):
        one_step()
    torch.cuda.synchronize()
    log(f"[bench] timing {args.steps} steps")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(args.steps):
        one_step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms_step = e0.elapsed_time(e1) / args.steps
    mlkv.profile_enable(args.steps * w.l)
    for _ in range(args.steps):
        one_step()
    torch.cuda.synchronize()
    n_launch, tot_ms, min_ms, max_ms = mlkv.profile_read()
    mlkv.profile_disable()
    avg = tot_ms * 1e-3 / n_launch
    if n_launch == args.steps:  # one launch reads each KV head once for all its layers
        attn_bytes = kv_bytes_once(w, np.full(B, w.ctx)) + qo_bytes
    else:
        attn_bytes = (kv_bytes + qo_bytes) / w.l
    achieved = attn_bytes / avg / 1e9
    per_seq = synth.step_bytes_per_sequence(w, S)
    floor = launch_floor(min(B * mp.layer_kv_count(0), 1 << 20))
    result = {
        "metric": "decode tokens/s at the largest batch whose 2048-token cache fits the GPU, "
                  "MLKV Pythia-160M shape",
        "value": round(B / (ms_step * 1e-3), 1),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) bf16 q/K/V generated on the device; no weights)",
        "config": {"workload": w.name, "l": w.l, "h": w.h, "m": w.m, "g": w.g, "head_dim": w.D,
                   "n_kv": w.n_kv, "batch": B, "ctx": w.ctx, "capacity": S,
                   "bytes_per_sequence": per_seq, "cache_bytes": int(cache.k.numel() * 4),
                   "kv_bytes_per_step": int(kv_bytes), "out_dtype": "bf16"},
        "max_batch": B,
        "step_gbs": round(step_total / (ms_step * 1e-3) / 1e9, 1),
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None,
                     "kernel": "step_kernel" if n_launch == args.steps else "attention_kernel",
                     "avg_launch_us": round(avg * 1e6, 2),
                     "min_launch_us": round(min_ms * 1e3, 2),
                     "max_launch_us": round(max_ms * 1e3, 2), "launches": n_launch,
                     "bytes_per_launch": int(attn_bytes), **floor,
                     "attainable_frac": attainable(attn_bytes, floor["launch_floor_us"]),
                     "read_reference": {"hbm_2GiB_gbs": hbm_ref},
                     "frac_of_hbm_read": round(achieved / hbm_ref, 4)},
    }
    if not args.no_cpu_baseline:
        log("[bench] cpu baseline (oracle)")
        # Bounded sample: whole decode steps of 4 sequences (rows copied back).
        sel = torch.arange(4, device=dev)
        q_h = mlkv.bf16_bits(q.index_select(1, sel))
        kn_h, vn_h = mlkv.bf16_bits(kn[:4]), mlkv.bf16_bits(vn[:4])
        # the sampled sequences' planes as plain token rows (mlkv_cache_read_rows)
        sub = mlkv.Cache(cache.k.index_select(1, sel).contiguous(),
                         cache.v.index_select(1, sel).contiguous())
        k_r, v_r = sub.read_rows()
        torch.cuda.synchronize()
        k_h, v_h = mlkv.bf16_bits(k_r), mlkv.bf16_bits(v_r)
        ctx_h = np.full(4, w.ctx, dtype=np.int32)
        import oracle

        kv_of, owner_of = oracle.map_uniform(w.l, w.h, w.m, w.g)
        threads = int(os.environ.get("OMP_NUM_THREADS", len(os.sched_getaffinity(0))))
        runs, spent = 0, 0.0
        while spent < 10.0 or runs == 0:
            k1, v1 = k_h.copy(), v_h.copy()
            ts = time.perf_counter()
            oracle.decode_step(q_h, k1, v1, kn_h, vn_h, kv_of, owner_of, ctx_h)
            spent += time.perf_counter() - ts
            runs += 1
        result["cpu_baseline"] = {
            "value": round(4 * runs / spent, 2), "unit": "tokens/s", "cores": threads,
            "kind": "oracle",
            "sample": f"{runs} whole decode step(s) of 4 sequences of the same workload "
                      f"(fp64 oracle), {spent:.1f} s"}
    print(json.dumps(result), flush=True)


def launch_floor(workgroups: int) -> dict:
    """The event-timing floor: the median event-pair duration of an empty
    kernel with the attention launch's workgroup count, launched back to back
    behind a GPU sleep (as the timed attention launches are)."""
    import torch
    import paper_2406_09297_amd as mlkv

    torch.cuda.synchronize()
    torch.cuda._sleep(SLEEP_CYCLES // 4)
    return {"launch_floor_us": round(mlkv.profile_launch_floor(workgroups, 256, 100) * 1e3, 3)}


def read_reference(bytes_per_launch: int, hbm_bytes: int = 2 << 30, cold_reps: int = 0) -> dict:
    """Achievable read rates, timed like the attention launches (event pairs
    recorded with each dispatch): a plain streaming read of the same bytes as
    one attention launch, warm in the caches (median of 20 back-to-back
    launches) and, with cold_reps, cold (the median of that many launches,
    each after the same 1 GiB flush read as the cold attention launches), and
    of a 2 GiB buffer, eight times the Infinity Cache (HBM)."""
    import torch
    import paper_2406_09297_amd as mlkv

    out = {}
    same = torch.ones((int(bytes_per_launch) + 16 + 15) // 16 * 4, dtype=torch.int32, device="cuda")
    mlkv.profile_read_bandwidth(same, reps=3)  # warm
    out["same_bytes_warm_gbs"] = round(mlkv.profile_read_bandwidth(same, reps=20)[0], 1)
    if cold_reps:
        flush = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        sink = torch.zeros((), device="cuda")
        cold = []
        for _ in range(cold_reps):
            flush_caches(flush, sink)
            cold.append(mlkv.profile_read_bandwidth(same, reps=1)[0])
        out["same_bytes_cold_gbs"] = round(float(np.median(cold)), 1)
        del flush
    del same
    if hbm_bytes:
        big = torch.ones(hbm_bytes // 4, dtype=torch.int32, device="cuda")
        out["hbm_2GiB_gbs"] = round(mlkv.profile_read_bandwidth(big, reps=5)[0], 1)
        del big
    torch.cuda.empty_cache()
    return out


def attainable(bytes_per_launch: float, floor_us: float) -> float:
    """Highest fraction of the HBM peak a launch timed this way can show:
    its bytes at peak rate plus the empty-launch floor."""
    t_peak = bytes_per_launch / (HBM_PEAK_GBS * 1e3)  # microseconds
    return round(t_peak / (t_peak + floor_us), 4)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default=DEFAULT_WORKLOAD)
    ap.add_argument("--map", default=None,
                    help="m,g of a map-sweep workload (default: its last point)")
    ap.add_argument("--long-context", default="mlkv4_b8_long",
                    help="second decode workload reported in the same line ('none' to skip)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--rotary-dims", type=int, default=0,
                    help="rotate the newest token's queries and keys inside the step "
                         "(GPT-NeoX rotary embedding; Pythia-160M: 16)")
    ap.add_argument("--rotary-base", type=float, default=10000.0)
    ap.add_argument("--batch", type=int, default=0,
                    help="model workload: batch size other than the workload's")
    ap.add_argument("--no-graph", action="store_true",
                    help="model workload: time eager launches only (default: graph replays)")
    ap.add_argument("--no-next-rows", action="store_true",
                    help="default workload: skip the prefill and model-step objects of the line")
    ap.add_argument("--pmc-pass", action="store_true",
                    help="for rocprofv3 --pmc runs: a 256 MiB reference copy, then a few steps")
    args = ap.parse_args()

    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only; the decode path is "
                                   "single-GPU (multi-GPU sharding is a design note, not built)",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    import synth
    import paper_2406_09297_amd as mlkv

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    torch.cuda.set_device(0)
    w = synth.get_workload(args.workload)
    if w.B == 0:  # batch sized at run time: the capacity experiment
        if args.map:
            m, g = (int(x) for x in args.map.split(","))
            w = w.with_map(m, g)
        run_capacity(args, w)
        return
    if w.T > 1:
        run_prefill(args, w)
        return
    if w.d_ff > 0:
        if args.map:
            m, g = (int(x) for x in args.map.split(","))
            w = w.with_map(m, g)
        elif w.sweep:
            m, g = w.sweep[-1]
            w = w.with_map(m, g)
        if args.batch:
            import dataclasses

            w = dataclasses.replace(w, B=args.batch, name=f"{w.name}-b{args.batch}")
        run_model(args, w)
        return
    if args.map:
        m, g = (int(x) for x in args.map.split(","))
        w = w.with_map(m, g)
    elif w.sweep:
        m, g = w.sweep[-1]
        w = w.with_map(m, g)
    result = measure_decode(args, w, dev, headline=True)
    if result is None:  # counter pass
        return
    extra = args.long_context
    if extra and extra != "none" and extra != w.name and not args.map:
        wl = synth.get_workload(extra)
        sub = measure_decode(args, wl, dev, headline=False)
        result["long_context"] = sub
    if w.name == DEFAULT_WORKLOAD and not args.map and not args.no_next_rows:
        # The rows after the decode path, timed in the same run: the causal
        # prefill of a 2000-token prompt and the whole-model decode step
        # (fewer steps; the line's CPU baseline is the decode step's).
        import copy

        sub_args = copy.copy(args)
        sub_args.no_cpu_baseline = True
        sub_args.steps = max(1, min(args.steps, 20))
        sub_args.warmup = max(1, min(args.warmup, 3))
        pw = synth.get_workload("prefill_b8_2000")
        mw = synth.get_workload("model_b8")
        if mw.sweep:
            mw = mw.with_map(*mw.sweep[-1])
        result["next_rows"] = {"prefill": run_prefill(sub_args, pw, emit=False),
                               "model_step": run_model(sub_args, mw, emit=False)}
    print(json.dumps(result), flush=True)


def flush_caches(flush, sink):
    """Evict the 256 MB Infinity Cache: a 1 GiB read (clean lines, no
    write-back) through a plain reduction on the current stream."""
    sink += flush.sum()


def measure_decode(args, w, dev, headline: bool):
    """The decode step of workload w: timed cold-start steps (value), warm
    back-to-back steps, and the attention launches (with their merge kernel
    when one follows) timed per launch by the library's event pairs, cold and
    in the warm step order.  Returns the JSON object (None for a counter pass)."""
    import torch
    import synth
    import paper_2406_09297_amd as mlkv

    log(f"[bench] workload {w.name}: generating inputs")
    inp = synth.step_inputs(w, fill=0)
    S = inp["capacity"]
    mp = mlkv.Map.uniform(w.l, w.h, w.m, w.g)
    cache = mlkv.Cache.empty(w.n_kv, w.B, S, w.D, dev)
    log("[bench] uploading")
    for kv in range(w.n_kv):
        cache.load_rows(inp["k_cache"][kv:kv + 1], inp["v_cache"][kv:kv + 1], (kv, kv + 1))
    q = mlkv.bf16_tensor(inp["q"], dev)
    kn = mlkv.bf16_tensor(inp["k_new"], dev)
    vn = mlkv.bf16_tensor(inp["v_new"], dev)
    ctx = torch.from_numpy(inp["ctx"]).to(dev)
    out = torch.empty((w.l, w.B, w.h, w.D), dtype=torch.float32, device=dev)
    ws = mlkv.workspace(mp, w.B, S, w.D, dev, rotary_dims=args.rotary_dims)
    ws_attn = mlkv.workspace(mp, w.B, S, w.D, dev)  # for single-layer calls
    max_len = int(inp["ctx"].max()) + 1
    stream = torch.cuda.current_stream()

    kv_count = [mp.layer_kv_count(n) for n in range(w.l)]
    owned = [mp.layer_owned(n)[1] for n in range(w.l)]
    per_layer = step_bytes(w, inp["ctx"], kv_count, owned)
    step_total = sum(sum(x.values()) for x in per_layer)
    kv_total = sum(x["kv"] for x in per_layer)
    attn_bytes = float(np.mean([x["kv"] + x["q"] + x["out"] for x in per_layer]))

    def one_step():
        mlkv.decode_step(q, kn, vn, cache, mp, ctx, out, max_len_hint=max_len, ws=ws,
                         rotary_dims=args.rotary_dims, rotary_base=args.rotary_base)

    if args.pmc_pass:
        # Counter pass: two plain copies of 256 MiB (a device-to-device copy
        # and an elementwise negation, each reading and writing 256 MiB once)
        # calibrate FETCH_SIZE / WRITE_SIZE; then steps in the benchmark's
        # launch configuration.
        src = torch.ones(REF_COPY_BYTES // 4, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.neg(src, out=dst)
        for _ in range(3):
            one_step()
        torch.cuda.synchronize()
        log("[bench] pmc pass done")
        return None

    log(f"[bench] warmup {args.warmup}")
    for _ in range(args.warmup):
        one_step()
    torch.cuda.synchronize()

    flush = torch.ones(1 << 28, dtype=torch.float32, device=dev)
    sink = torch.zeros((), device=dev)

    # (1) Cold-start steps (value): the Infinity Cache is flushed before each
    # step, so every step starts with its inputs in HBM only; inside a step
    # the layers sharing a KV head meet it where the previous layer left it,
    # as they would in a model.  An event pair per step; the flushes are
    # outside the pairs.  The host enqueues all of it behind a GPU sleep.
    log(f"[bench] timing {args.steps} cold-start steps")
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(args.steps)]
    torch.cuda.synchronize()
    torch.cuda._sleep(SLEEP_CYCLES)
    for e0, e1 in evs:
        flush_caches(flush, sink)
        e0.record(stream)
        one_step()
        e1.record(stream)
    torch.cuda.synchronize()
    step_ms = np.array([e0.elapsed_time(e1) for e0, e1 in evs])
    ms_step = float(step_ms.mean())

    # (2) Warm back-to-back steps: the whole cache of this workload may stay
    # in the Infinity Cache between steps (effective bandwidth, not HBM).
    log(f"[bench] timing {args.steps} warm back-to-back steps")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(args.steps):
        one_step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms_warm = e0.elapsed_time(e1) / args.steps

    # (3) Per launch, cold: a flush before every layer's attention as its own
    # call (mlkv_decode_attention; the pair brackets the merge kernel too when
    # one follows): the roofline's figure of the one-layer kernel.
    log("[bench] cold attention launches")
    lens_attn = (ctx + 1).to(torch.int32)
    out_l = torch.empty((w.B, w.h, w.D), dtype=torch.float32, device=dev)
    reps = max(3 * w.l, min(args.steps, 10 * w.l))
    mlkv.profile_enable(reps)
    for i in range(reps):
        n = i % w.l
        flush_caches(flush, sink)
        mlkv.decode_attention(n, q[n], cache, mp, lens_attn, out_l, max_len_hint=max_len,
                              ws=ws_attn)
    torch.cuda.synchronize()
    c_n, _, c_min, c_max = mlkv.profile_read()
    c_dur = mlkv.profile_durations(c_n)
    mlkv.profile_disable()
    # ... and before every step: its own launches, one where all layers share it.
    s_reps = min(args.steps, 30)
    mlkv.profile_enable(s_reps * w.l)
    for _ in range(s_reps):
        flush_caches(flush, sink)
        one_step()
    torch.cuda.synchronize()
    s_n, s_tot, s_min, s_max = mlkv.profile_read()
    mlkv.profile_disable()
    del flush
    torch.cuda.empty_cache()
    c_avg = float(c_dur.mean()) * 1e-3
    achieved = attn_bytes / c_avg / 1e9

    # (4) Per launch, warm: the library's pairs around each layer's attention
    # inside back-to-back steps (chunks of ten steps enqueued behind a GPU
    # sleep, so no interval holds host launch latency).
    log("[bench] warm attention launches (event pairs)")
    mlkv.profile_enable(args.steps * w.l)
    torch.cuda.synchronize()
    done = 0
    while done < args.steps:
        n = min(10, args.steps - done)
        torch.cuda._sleep(SLEEP_CYCLES)
        for _ in range(n):
            one_step()
        torch.cuda.synchronize()
        done += n
    n_launch, w_tot, _, _ = mlkv.profile_read()
    mlkv.profile_disable()
    w_avg = w_tot * 1e-3 / n_launch
    # A step in one launch reads each cached byte once for all its layers.
    once = kv_bytes_once(w, inp["ctx"]) + sum(x["q"] + x["out"] for x in per_layer)
    w_bytes = once if n_launch == args.steps else attn_bytes
    s_bytes = once if s_n == s_reps else attn_bytes
    s_avg = s_tot * 1e-3 / s_n

    workgroups, max_parts = mp.plan(0, w.B, S, w.D, max_len)
    floor = launch_floor(workgroups)
    ref = read_reference(int(attn_bytes), cold_reps=15)
    p10, p50, p90 = (float(np.percentile(c_dur, pq)) for pq in (10, 50, 90))
    gbs = step_total / (ms_step * 1e-3) / 1e9
    warm_gbs = step_total / (ms_warm * 1e-3) / 1e9
    merge_kernel = mp.plan_merge_kernel(0, w.B, S, w.D, max_len)
    kernel = "attention_kernel" + (" + combine_kernel" if merge_kernel else "")
    roofline = {
        "bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
        "frac": round(achieved / HBM_PEAK_GBS, 4),
        "traffic": measured_traffic(w.name) if not args.rotary_dims else None,
        "kernel": kernel,
        "avg_launch_us": round(c_avg * 1e6, 3),
        "min_launch_us": round(c_min * 1e3, 3), "max_launch_us": round(c_max * 1e3, 3),
        "p10_p50_p90_launch_us": [round(p10 * 1e3, 3), round(p50 * 1e3, 3), round(p90 * 1e3, 3)],
        "launches": c_n, "bytes_per_launch": int(attn_bytes),
        "cache_state": "Infinity Cache flushed (1 GiB read) before each launch: K/V from HBM",
        "step_launch": {"kernel": "step_kernel" if s_n == s_reps else kernel,
                        "avg_launch_us": round(s_avg * 1e6, 3),
                        "min_launch_us": round(s_min * 1e3, 3),
                        "max_launch_us": round(s_max * 1e3, 3),
                        "achieved": round(s_bytes / s_avg / 1e9, 1),
                        "frac": round(s_bytes / s_avg / 1e9 / HBM_PEAK_GBS, 4),
                        "launches": s_n, "bytes_per_launch": int(s_bytes),
                        "cache_state": "what the timed step launches, Infinity Cache flushed "
                                       "before each step; the figures above are of one layer's "
                                       "attention as a call of its own"},
        "warm": {"avg_launch_us": round(w_avg * 1e6, 3),
                 "achieved": round(w_bytes / w_avg / 1e9, 1),
                 "frac": round(w_bytes / w_avg / 1e9 / HBM_PEAK_GBS, 4),
                 "launches": n_launch, "bytes_per_launch": int(w_bytes),
                 "cache_state": "the step's own launches, back-to-back steps (the Infinity "
                                "Cache may hold the rows: effective bandwidth, not HBM)"},
        **floor,
        "attainable_frac": attainable(attn_bytes, floor["launch_floor_us"]),
        "read_reference": ref,
        "frac_of_hbm_read": round(achieved / ref["hbm_2GiB_gbs"], 4),
        "frac_of_same_bytes_cold_read": round(achieved / ref["same_bytes_cold_gbs"], 4),
    }
    result = {
        "metric": "decode-attention HBM GB/s (% of peak) + decode steps/s, MLKV Pythia-160M shape",
        "value": round(gbs, 2),
        "unit": "GB/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 5),
        "steps_per_s": round(1e3 / ms_step, 1),
        "pct_of_hbm_peak": round(100 * achieved / HBM_PEAK_GBS, 2),
        "step_pct_of_hbm_peak": round(100 * gbs / HBM_PEAK_GBS, 2),
        "step_bytes_once": int(once), "step_once_gbs": round(once / (ms_step * 1e-3) / 1e9, 2),
        "value_note": "value counts every layer's read of its KV heads; the step reads a head "
                      "shared by several layers once for all of them, so value may exceed the "
                      "HBM peak: step_once_gbs counts each cached byte once",
        "kv_gbs": round(kv_total / (ms_step * 1e-3) / 1e9, 2),
        "step_timing": "cold start: Infinity Cache flushed before each step (outside the "
                       "timed pairs); K/V of each step from HBM",
        "warm_steps": {"ms_per_step": round(ms_warm, 5), "steps_per_s": round(1e3 / ms_warm, 1),
                       "gbs": round(warm_gbs, 2),
                       "note": "back-to-back steps: this workload's cache may stay in the "
                               "256 MB Infinity Cache between steps (effective bandwidth)"},
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) bf16 q/K/V; no weights)",
        "config": {"workload": w.name, "l": w.l, "h": w.h, "m": w.m, "g": w.g, "head_dim": w.D,
                   "batch": w.B, "ctx": w.ctx if w.ctx is not None else list(w.ctx_range),
                   "ctx_sum": int(inp["ctx"].sum()), "capacity": S,
                   "bytes_per_step": int(step_total), "kv_bytes_per_step": int(kv_total),
                   "workgroups_layer0": workgroups, "rotary_dims": args.rotary_dims},
        "roofline": roofline,
    }
    if headline and not args.no_cpu_baseline:
        log("[bench] cpu baseline (oracle)")
        import oracle

        kv_of, owner_of = oracle.map_uniform(w.l, w.h, w.m, w.g)
        result["cpu_baseline"] = cpu_baseline(w, inp, kv_of, owner_of, step_total,
                                              rotary=(args.rotary_dims, args.rotary_base))
    if not headline:
        for k in ("metric", "n_gpus", "steps", "warmup", "higher_is_better", "scaling",
                  "vs_baseline", "dtype", "data"):
            result.pop(k, None)
    return result


if __name__ == "__main__":
    main()
