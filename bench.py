"""Verify-step throughput of the tree-verification path on one MI355X.

    python bench.py [--steps K] [--warmup W] [--workload qwen3-8b] [--cpu-seconds S]

A step is one whole verification pass over one batch of synthetic input at
the Qwen3-8B shape (36 layers, 32 query / 8 KV heads, head_dim 128, 4096
committed prefix rows, 64-node trie, hidden 4096, vocabulary 151936, bf16):

  host   ooo_pack_tree of the step's candidates (hint, FSM chain, 2 retrieved)
  copy   H2D of the packed trie
  graph  36 x ooo_tree_attn, bracketed by HIP events on its stream
  eager  ooo_lmhead_argmax, bracketed by HIP events on its stream
  graph  ooo_accept, ooo_kv_compact, D2H of (L, bonus, path)
  host   stream synchronise and read the accepted length (the next step's
         candidates depend on it in a real decode loop)

All inputs are resident in HBM before timing starts.  The nodes' K/V rows
sit in the cache scratch rows [P, P+N) of every layer; in a model the
projection kernels rewrite them each step, which is outside this path, so
the rows that compaction leaves there serve as the next step's node rows.
Prints one JSON line.
The roofline object covers ooo_tree_attn, the kernel pair that takes most of
a step; the LM head has one of its own.  --calibrate-copy-mib M adds one
plain device copy of M MiB after setup, outside the timed steps, so that
hardware byte counters read under a profiler can be scaled by what they
report for a copy of known size.
"""

from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import platform
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
MFMA_PEAK_TFLOPS = 2500.0  # dense bf16 matrix cores
FP32_PEAK_TFLOPS = 157.3   # fp32 (the tiny fp32 workload runs on the vector units)
METRIC = "verify steps/s + tree-attn/LM-head HBM GB/s, Qwen3-8B shape, 64-node trie, 4k ctx"


def attention_bytes(cfg, N):
    """Algorithmic HBM bytes of one layer: K/V prefix + K/V of the nodes + Q + O."""
    e = cfg.elt_bytes
    kv = 2 * cfg.n_kv_heads * (cfg.prefix_len + N) * cfg.head_dim * e
    qo = 2 * N * cfg.n_q_heads * cfg.head_dim * e
    return kv + qo


def lmhead_bytes(cfg, N):
    """W + X + greedy ids and max logits."""
    e = cfg.elt_bytes
    return cfg.vocab * cfg.hidden * e + N * cfg.hidden * e + N * 8


# The paper's own end-to-end numbers for context (Section 6.1, Table 2): they
# measure whole requests on other hardware, so they are reported beside the
# bench line, never as its baseline.
PAPER_CONTEXT = {
    "speedup_over_autoregressive": "2.46x-5.34x (21 target/benchmark cells, mean 3.89x)",
    "qwen3_8b_api_bank": {"mean_accepted_tokens_per_call": 8.35, "tokens_per_s": 207.09, "speedup": 5.34},
    "hardware": "H100-80GB, greedy, batch 1, Qwen3 targets in BF16 under HF Transformers, sidecar on a second GPU",
    "source": "Section 6.1, Table 2",
    "note": "end-to-end request latency including drafting; context only, not the target of this bench",
}
PAPER_MAT_QWEN3_8B = 8.35  # tokens committed per verify call, Qwen3-8B on API-Bank (Table 2)


# The other path workloads, timed kernel by kernel in the default run.
SECONDARY_WORKLOADS = ("qwen3-0.6b", "qwen2.5-32b", "llama3.1-8b-decode")


def kernel_record(cfg, N, attn_call_us, lm_us):
    """Roofline figures of one tree-attention call and one LM head at a
    workload's shapes (same byte and flop counts as the headline line)."""
    a_bytes = attention_bytes(cfg, N)
    a_flops = 4.0 * cfg.n_q_heads * N * cfg.prefix_len * cfg.head_dim
    peak = MFMA_PEAK_TFLOPS if cfg.dtype == "bf16" else FP32_PEAK_TFLOPS
    mfma_bound = a_flops / a_bytes > peak * 1e12 / (HBM_PEAK_GBS * 1e9)
    a_gbs = a_bytes / (attn_call_us * 1e-6) / 1e9
    a_tflops = a_flops / (attn_call_us * 1e-6) / 1e12
    lm_gbs = lmhead_bytes(cfg, N) / (lm_us * 1e-6) / 1e9
    return {"trie_nodes": N, "prefix_len": cfg.prefix_len,
            "attention_us_per_call": round(attn_call_us, 3),
            "attention_bound": "mfma" if mfma_bound else "hbm",
            "attention_frac": round(a_tflops / peak if mfma_bound else a_gbs / HBM_PEAK_GBS, 4),
            "attention_hbm_frac": round(a_gbs / HBM_PEAK_GBS, 4),
            "attention_mfma_frac": round(a_tflops / peak, 4),
            "lmhead_us": round(lm_us, 2), "lmhead_hbm_frac": round(lm_gbs / HBM_PEAK_GBS, 4)}


def tp8_shard_config():
    """One GPU's share of the Qwen3-8B shape under 8-way tensor parallelism
    over KV heads and vocabulary rows: 1 KV head with its 4 query heads, and
    1/8 of the LM-head rows (the trie is the full step's)."""
    import dataclasses

    from paper_2608_00814_amd import workload as wl
    q8b = wl.CONFIGS["qwen3-8b"]
    return dataclasses.replace(q8b, n_q_heads=q8b.n_q_heads // 8, n_kv_heads=q8b.n_kv_heads // 8,
                               vocab=q8b.vocab // 8)


def secondary_rates(name, dev, reps: int = 10):
    """Tree attention and LM head at another workload's shapes: the
    workload's own trie, K/V ~ N(0, 1) and LM-head weights ~ N(0, 0.02)
    from a seeded device generator (the recipe's distributions without the
    host-side generation of whole caches), enough distinct layer caches to
    cycle past the 256 MiB last-level cache, one graph of those attention
    calls, then the LM head; medians over reps."""
    import torch

    from paper_2608_00814_amd import workload as wl
    from paper_2608_00814_amd.step import VerifyRunner

    cfg = wl.CONFIGS[name] if isinstance(name, str) else name
    tdt = torch.bfloat16
    P = cfg.prefix_len
    runner = VerifyRunner(cfg.n_layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden, cfg.vocab,
                          cfg.max_nodes, cfg.max_depth, tdt, dev, max_prefix=P)
    cand = wl.candidates_for(cfg, 0, 0)
    runner.pack(cand.root_token, *cand.csr())
    N = runner.n_nodes
    runner.ensure_workspace(P)
    gen = torch.Generator(device=dev)
    gen.manual_seed(2608)
    per_layer = 2 * cfg.n_kv_heads * cfg.cap * cfg.head_dim * 2
    L = max(2, min(256, -(-(640 << 20) // per_layer)))
    shp = (cfg.n_kv_heads, cfg.cap, cfg.head_dim)
    k = torch.empty((L,) + shp, dtype=tdt, device=dev)
    v = torch.empty((L,) + shp, dtype=tdt, device=dev)
    for l in range(L):
        k[l].copy_(torch.randn(shp, generator=gen, device=dev))
        v[l].copy_(torch.randn(shp, generator=gen, device=dev))
    q = torch.randn((N, cfg.n_q_heads, cfg.head_dim), generator=gen, device=dev).to(tdt)
    w = (torch.randn((cfg.vocab, cfg.hidden), generator=gen, device=dev) * 0.02).to(tdt)
    runner.set_weight(w)
    del w
    hidden = torch.randn((N, cfg.hidden), generator=gen, device=dev).to(tdt)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()  # default priority
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    attn_us, lm_us = [], []
    with torch.cuda.stream(stream):
        runner.upload_tree()

        def attend():
            for l in range(L):
                runner.attention(l % cfg.n_layers, q, k[l], v[l], P)

        attend()
        runner.lm_head(hidden)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            attend()
        for _ in range(reps):
            ev[0].record(stream)
            graph.replay()
            ev[1].record(stream)
            runner.lm_head(hidden)
            ev[2].record(stream)
            stream.synchronize()
            attn_us.append(1e3 * ev[0].elapsed_time(ev[1]) / L)
            lm_us.append(1e3 * ev[1].elapsed_time(ev[2]))
    rec = kernel_record(cfg, N, float(np.median(attn_us)), float(np.median(lm_us)))
    rec["layer_caches_cycled"] = L
    del graph, k, v, q, hidden, runner
    torch.cuda.empty_cache()
    return rec


def step_time_stats(step_s):
    """Median and 10th/90th percentiles of per-step wall times (ms)."""
    a = np.asarray(step_s, dtype=np.float64) * 1e3
    return {"median_ms": round(float(np.median(a)), 4), "p10_ms": round(float(np.percentile(a, 10)), 4),
            "p90_ms": round(float(np.percentile(a, 90)), 4)}


def host_cpu():
    """CPU model (from /proc/cpuinfo) and the cores this process may use."""
    model = platform.processor() or "unknown"
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return model, len(os.sched_getaffinity(0))


def tokens_at_mat(steps_per_s: float, mat: float = PAPER_MAT_QWEN3_8B):
    """Tokens/s if every verify step committed ``mat`` tokens (the paper's
    measured acceptance instead of the planted one)."""
    return {"mean_accepted_tokens_per_call": mat, "tokens_per_s": round(steps_per_s * mat, 1),
            "source": "Section 6.1, Table 2 (Qwen3-8B, API-Bank)"}


def copy_bandwidth_gbs(dev, mib: int = 1024, reps: int = 10) -> float:
    """Read + write GB/s of a plain device copy of ``mib`` MiB (context for
    the roofline fraction: what a copy kernel reaches on this GPU)."""
    import torch
    src = torch.empty(mib << 18, dtype=torch.float32, device=dev).fill_(1.0)
    dst = torch.empty_like(src)
    for _ in range(2):
        dst.copy_(src)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    sec = e0.elapsed_time(e1) * 1e-3 / reps
    del src, dst
    return 2.0 * (mib << 20) / sec / 1e9


def calibration_copy(mib: int, dev) -> None:
    """One plain elementwise copy that reads and writes ``mib`` MiB each (the
    byte counters' calibration kernel); nothing when mib is 0."""
    if mib <= 0:
        return
    import torch
    src = torch.ones(mib << 18, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    torch.add(src, 1.0, out=dst)
    torch.cuda.synchronize()
    del src, dst


def _source_digest(path: str) -> str:
    """sha256 prefix of a source file with comments and whitespace removed."""
    text = open(os.path.join(ROOT, path)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    text = re.sub(r"//[^\n]*", "", text)
    return hashlib.sha256(" ".join(text.split()).encode()).hexdigest()[:16]


def time_hint_merge(cfg, cand_sets, reps: int = 200):
    """Host time of one retrieval round's lane filling (ooo_hint_merge on a
    request-level hint bank of eight 512-token views), per call.  Outside the
    verify step: it runs at retrieval rounds, before ooo_pack_tree."""
    from paper_2608_00814_amd import ooo
    from paper_2608_00814_amd import workload as wl
    banks = [wl.hint_bank_for(cfg, s, c) for s, c in enumerate(cand_sets)]
    natives = []
    for c, hb in zip(cand_sets, banks):
        seqs = c.seqs[1:]
        offs = np.zeros(len(seqs) + 1, np.int32)
        for i, q in enumerate(seqs):
            offs[i + 1] = offs[i] + len(q)
        toks = np.array([t for q in seqs for t in q], dtype=np.int32)
        natives.append((toks, offs, len(c.seqs)))
        r = ooo.hint_merge(hb.bank, hb.eos, hb.committed, toks, offs, len(c.seqs), 7, cfg.max_depth)
        lanes = [r["tokens"][r["offsets"][i]:r["offsets"][i + 1]].tolist() for i in range(r["n_out"])]
        assert lanes == [list(q[:cfg.max_depth]) for q in c.seqs], "hint bank must reproduce the candidate lanes"
    t0 = time.perf_counter()
    for i in range(reps):
        hb, (toks, offs, nl) = banks[i % len(banks)], natives[i % len(banks)]
        ooo.hint_merge(hb.bank, hb.eos, hb.committed, toks, offs, nl, 7, cfg.max_depth)
    return 1e6 * (time.perf_counter() - t0) / reps, int(banks[0].bank.size)


def recorded_traffic(workload: str, entry: str):
    """HBM bytes per launch that the committed counter profile records for
    ``entry``, or None when there is none for this workload or the kernel
    sources have changed since it was taken."""
    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{workload}.json")
    if not os.path.exists(path):
        return None
    rec = json.load(open(path)).get(entry)
    if not rec or any(_source_digest(f) != d for f, d in rec["sources"].items()):
        return None
    return int(rec["bytes_per_launch"])


# Kernels whose counters make up each entry point's traffic, and the sources
# whose digests decide whether a recorded profile still describes them.
TRAFFIC_ENTRIES = {
    "ooo_tree_attn": (("tree_attn_bf16_kernel", "tree_attn_combine_kernel"),
                      ("paper_2608_00814_amd/csrc/tree_attn.hip", "paper_2608_00814_amd/csrc/device_common.h")),
    "ooo_lmhead_argmax": (("lmhead_bf16_kernel", "lmhead_finalize_kernel"),
                          ("paper_2608_00814_amd/csrc/lmhead.hip", "paper_2608_00814_amd/csrc/stream_core.h",
                           "paper_2608_00814_amd/csrc/device_common.h")),
}
# The projection kernels of one fused decoder layer (ModelRunner.forward):
# four streaming products (qkv, o, gate+up, down), then the qkv epilogue
# (norms, rotation, cache writes), two residual-add + RMSNorm epilogues and,
# where gate+up goes through partial sums, the SwiGLU reduce; by whole columns
# it is one kernel of its own.  Count per layer, and the sources they are built
# from.
MODEL_PROJECTION_KERNELS = {"linear_bf16_kernel": 4, "linear_add_rmsnorm_kernel": 2,
                            "linear_qk_norm_rope_kernel": 1, "linear_reduce_kernel": 1}
MODEL_PROJECTION_KERNELS_COLUMNS = {"linear_bf16_kernel": 3, "linear_swiglu_kernel": 1,
                                    "linear_add_rmsnorm_kernel": 2, "linear_qk_norm_rope_kernel": 1}
MODEL_PROJECTION_SOURCES = ("paper_2608_00814_amd/csrc/linear.hip", "paper_2608_00814_amd/csrc/stream_core.h",
                            "paper_2608_00814_amd/csrc/rope.h", "paper_2608_00814_amd/csrc/runs.h",
                            "paper_2608_00814_amd/csrc/device_common.h")
CALIBRATION_KERNEL = "CUDAFunctorOnSelf_add<float>"  # torch.add(src, 1.0, out=dst) of --calibrate-copy-mib


def _short_kernel_name(name: str) -> str:
    """'void ooo::(anonymous namespace)::k<1, 2>(args)' -> 'ooo::k<1, 2>'."""
    name = name.replace("(anonymous namespace)::", "")
    if name.startswith("void "):
        name = name[5:]
    depth = 0
    for i, ch in enumerate(name):
        if ch == "<":
            depth += 1
        elif ch == ">":
            depth -= 1
        elif ch == "(" and depth == 0:
            return name[:i]
    return name


def counter_means(csv_path: str, counter: str):
    """Mean value (KiB) of one rocprofv3 --pmc counter per dispatch, by
    kernel (short name)."""
    import csv
    sums, counts = {}, {}
    for row in csv.DictReader(open(csv_path)):
        if row["Counter_Name"] != counter:
            continue
        k = _short_kernel_name(row["Kernel_Name"])
        sums[k] = sums.get(k, 0.0) + float(row["Counter_Value"])
        counts[k] = counts.get(k, 0) + 1
    return {k: sums[k] / counts[k] for k in sums}


def traffic_record(workload: str, fetch_csv: str, write_csv: str, calibrate_mib: int) -> dict:
    """HBM bytes per launch of each entry point from one FETCH_SIZE and one
    WRITE_SIZE profile of the same bench run.  Each counter is scaled by
    what it reads for the calibration kernel, which reads and writes
    calibrate_mib MiB; the sources' digests are stored with the numbers.
    For a full-model workload the one entry is "projections": the bytes of
    every projection kernel of one verify step (all layers)."""
    fetch, write = counter_means(fetch_csv, "FETCH_SIZE"), counter_means(write_csv, "WRITE_SIZE")
    cal = [k for k in fetch if CALIBRATION_KERNEL in k]
    if len(cal) != 1 or cal[0] not in write:
        raise ValueError("the profiles hold no single calibration copy (bench.py --calibrate-copy-mib)")
    fs, ws = calibrate_mib * 1024.0 / fetch[cal[0]], calibrate_mib * 1024.0 / write[cal[0]]
    rec = {"workload": workload, "fetch_scale": round(fs, 5), "write_scale": round(ws, 5)}
    from paper_2608_00814_amd import model_workload as mw
    if workload in mw.MODEL_CONFIGS:
        n_layers = mw.MODEL_CONFIGS[workload].n_layers
        kernels = {}
        columns = any("linear_swiglu_kernel" in k for k in fetch)
        for part, per_layer in (MODEL_PROJECTION_KERNELS_COLUMNS if columns else MODEL_PROJECTION_KERNELS).items():
            ks = [k for k in fetch if part in k]
            if len(ks) != 1:
                raise ValueError(f"expected one instantiation of {part} in the profile, found {ks}")
            kernels[ks[0]] = [fetch[ks[0]], write.get(ks[0], 0.0), per_layer * n_layers]
        rec["projections"] = {
            "bytes_per_launch": int(round(sum((f * fs + w * ws) * 1024 * n for f, w, n in kernels.values()))),
            "kernels": kernels,
            "sources": {f: _source_digest(f) for f in MODEL_PROJECTION_SOURCES},
        }
        return rec
    for entry, (parts, sources) in TRAFFIC_ENTRIES.items():
        ks = sorted(k for k in fetch if any(p in k for p in parts))
        if not ks:
            continue
        rec[entry] = {
            "bytes_per_launch": int(round(sum((fetch[k] * fs + write.get(k, 0.0) * ws) * 1024 for k in ks))),
            "kernels": {k: [fetch[k], write.get(k, 0.0)] for k in ks},
            "sources": {f: _source_digest(f) for f in sources},
        }
    return rec


def _blas_limit(cores: int):
    """Context manager pinning NumPy's BLAS pool to ``cores`` threads (a
    no-op without threadpoolctl)."""
    try:
        from threadpoolctl import threadpool_limits
        return threadpool_limits(limits=cores)
    except Exception:  # pragma: no cover
        import contextlib
        return contextlib.nullcontext()


def cpu_baseline(cfg, seconds: float):
    """Time the CPU reference on whole verification steps of the same
    workload until about ``seconds`` have passed (at least one step), with
    the BLAS pool on every core the process may use."""
    model, cores = host_cpu()
    with _blas_limit(cores):
        return _cpu_baseline(cfg, seconds, model, cores)


def _cpu_baseline(cfg, seconds: float, model: str, threads: int):
    from oracle import tree_verify as ov
    from paper_2608_00814_amd import workload as wl

    seed = 0
    cands = wl.candidates_for(cfg, seed, 0)
    tree = ov.pack_tree(cands.root_token, cands.seqs, cands.max_nodes, cands.max_depth)
    N = tree["n_nodes"]
    tau, _ = wl.designated_tokens(cfg, seed, 0, cands, tree["token"], tree["parent"])
    w_st = wl.lm_head_weight(cfg, seed)
    x64 = wl.to_f64(wl.hidden_rows(cfg, seed, 0, w_st, tau, N), cfg.dtype)
    w64 = wl.to_f32(w_st, cfg.dtype)  # exact; the reference widens it to float64 chunk by chunk
    del w_st
    layers = []
    for l in range(cfg.n_layers):
        k, v = wl.layer_cache(cfg, seed, l, N)
        layers.append((wl.to_f64(wl.queries(cfg, seed, 0, l, N), cfg.dtype), wl.to_f64(k, cfg.dtype),
                       wl.to_f64(v, cfg.dtype)))
    steps = 0
    t0 = time.perf_counter()
    while True:
        res = ov.verify_step(cands.root_token, cands.seqs, cands.max_nodes, cands.max_depth, layers,
                             cfg.prefix_len, cfg.n_kv_heads, x64, w64)
        kc = [l[1] for l in layers]
        vc = [l[2] for l in layers]
        ov.kv_compact(kc + vc, cfg.prefix_len, res["path"])
        steps += 1
        el = time.perf_counter() - t0
        if el >= seconds:
            break
    return {"value": steps / el, "unit": "verify steps/s", "cores": threads, "kind": "oracle",
            "cpu_model": model,
            "sample": f"{steps} whole {cfg.name} verify step(s) (pack, {cfg.n_layers}-layer tree attention, "
                      f"LM head, accept, compact) in fp64 NumPy, {el:.1f} s, on {model} with the BLAS pool on "
                      f"the {threads} cores of the process affinity"}


MODEL_METRIC = "full-model verify steps/s, Qwen3-8B decoder (36 layers, random weights), 64-node trie, 4k ctx"


def model_cpu_baseline(mcfg, seconds: float):
    """The decoder reference on a bounded sample of the full-model step: one
    full-size layer over the step's trie (repeated until about ``seconds``
    have passed) plus one LM head and accept; the step time is scaled to all
    layers."""
    model_name, threads = host_cpu()
    with _blas_limit(threads):
        return _model_cpu_baseline(mcfg, seconds, model_name, threads)


def _model_cpu_baseline(mcfg, seconds: float, cpu_name: str, threads: int):
    from oracle import target_model as om
    from oracle import tree_verify as ov
    from paper_2608_00814_amd import model_workload as mw
    from paper_2608_00814_amd import workload as wl
    f64 = wl.bf16_to_f64
    seed = 0
    pcfg = wl.CONFIGS["qwen3-8b"]
    cands = wl.candidates_for(pcfg, seed, 0)
    tree = ov.pack_tree(cands.root_token, cands.seqs, mcfg.max_nodes, mcfg.max_depth)
    lw = om.LayerWeights(**{k: f64(v) for k, v in mw.layer_weights(mcfg, seed, 0).items()})
    shp = om.ModelShape(hidden=mcfg.hidden, n_q_heads=mcfg.n_q_heads, n_kv_heads=mcfg.n_kv_heads,
                        head_dim=mcfg.head_dim, intermediate=mcfg.intermediate, rope_theta=mcfg.rope_theta,
                        eps=mcfg.eps)
    k, v = mw.prefix_kv(mcfg, seed, 0)
    kc, vc = f64(k), f64(v)
    emb = mw.embedding(mcfg, seed)
    h = f64(emb[np.asarray(tree["token"])])
    del emb
    reps = 0
    t0 = time.perf_counter()
    while True:
        out = om.decoder_layer(h, lw, shp, kc, vc, mcfg.prefix_len, tree["parent"], tree["depth"])
        reps += 1
        el = time.perf_counter() - t0
        if el >= seconds:
            break
    t_layer = el / reps
    lm = mw.lm_head(mcfg, seed)
    t1 = time.perf_counter()
    x = om.rmsnorm(out["h"], f64(mw.final_norm(mcfg, seed)), mcfg.eps)
    g = ov.greedy_tokens(ov.lm_head_logits(x, _Widen(lm)))
    ov.accept_walk(tree["token"], tree["parent"], g["ids"])
    t_head = time.perf_counter() - t1
    step = mcfg.n_layers * t_layer + t_head
    return {"value": 1.0 / step, "unit": "verify steps/s", "cores": threads, "kind": "oracle",
            "cpu_model": cpu_name,
            "sample": f"{reps} full-size decoder layer(s) over the step's {tree['n_nodes']}-node trie "
                      f"({t_layer:.2f} s each) plus one LM head and accept ({t_head:.2f} s) in fp64 NumPy, "
                      f"scaled to {mcfg.n_layers} layers, on {cpu_name} with the BLAS pool on the {threads} "
                      f"cores of the process affinity"}


class _Widen:
    """bf16 table widened to float64 on indexing (row chunks of the LM head)."""

    def __init__(self, bits):
        self.bits, self.shape = bits, bits.shape

    def __getitem__(self, idx):
        from paper_2608_00814_amd import workload as wl
        return wl.bf16_to_f64(self.bits[idx])


def bench_model(args):
    """Full verify steps of a Qwen3-8B-shaped decoder (random weights): the
    decoder layers around the path, LM head, accept, compact."""
    import torch

    from paper_2608_00814_amd import model_workload as mw
    from paper_2608_00814_amd import ooo
    from paper_2608_00814_amd import workload as wl
    from paper_2608_00814_amd.model import ModelRunner

    ooo.lib()
    mcfg = mw.MODEL_CONFIGS[args.workload]
    dev = torch.device("cuda:0")
    P = mcfg.prefix_len
    t_setup = time.time()
    seed = 0
    layers = (mw.layer_weights(mcfg, seed, l) for l in range(mcfg.n_layers))  # uploaded one at a time
    runner = ModelRunner(mcfg, layers, mw.embedding(mcfg, seed), mw.final_norm(mcfg, seed), mw.lm_head(mcfg, seed),
                         dev)
    shp = (mcfg.n_layers, mcfg.n_kv_heads, mcfg.cap, mcfg.head_dim)
    k_cache = torch.empty(shp, dtype=torch.bfloat16, device=dev)
    v_cache = torch.empty(shp, dtype=torch.bfloat16, device=dev)
    for l in range(mcfg.n_layers):
        k, v = mw.prefix_kv(mcfg, seed, l)
        k_cache[l].copy_(torch.from_numpy(k.view(np.int16)).view(torch.bfloat16))
        v_cache[l].copy_(torch.from_numpy(v.view(np.int16)).view(torch.bfloat16))
    stream = torch.cuda.Stream()
    pcfg = wl.CONFIGS["qwen3-8b"]
    with torch.cuda.stream(stream):
        # the model's own greedy continuation of the root (planted into each
        # step's first candidate, to a depth drawn like the path workload's)
        root = wl.candidates_for(pcfg, seed, 0).root_token
        rs = np.random.default_rng(1)

        def lanes(c, first):
            # the path workload's trie shape with `first` as its first lane
            # (the hint): the other lanes' prefixes shared with the hint follow
            hint = list(c.seqs[0])
            seqs = [first]
            for q in c.seqs[1:]:
                m = 0
                while m < min(len(q), len(hint)) and q[m] == hint[m]:
                    m += 1
                seqs.append(first[:m] + list(q[m:]))
            offs = np.zeros(len(seqs) + 1, np.int32)
            for i, q in enumerate(seqs):
                offs[i + 1] = offs[i] + len(q)
            return np.array([t for q in seqs for t in q], np.int32), offs

        # the model's own greedy continuation of the root, built in tries of
        # the same shape as the timed steps (so every row is computed exactly
        # as it will be there): the depth-k node of the first lane is node k
        c0 = wl.candidates_for(pcfg, 0, 0)
        lane_len = len(c0.seqs[0])
        filler = [int(t) for t in rs.integers(0, mcfg.vocab, size=lane_len)]
        chain = []
        for k in range(lane_len + 1):
            runner.pack(root, *lanes(c0, chain + filler[k:]), keep=False)
            runner.device_step(k_cache, v_cache, P, compact=False)
            stream.synchronize()
            chain.append(int(runner.vr.ids[k].item()))
        # variants: the greedy chain up to depth d, a wrong token, fresh tokens
        n_variants = 4
        cand_sets, depths = [], []
        for s in range(n_variants):
            d = int(rs.integers(4, min(mcfg.max_depth, lane_len) + 1))
            first = chain[:d] + [(chain[d] + 1) % mcfg.vocab]
            first += [int(t) for t in rs.integers(0, mcfg.vocab, size=lane_len - len(first))]
            cand_sets.append(lanes(c0, first))
            depths.append(d)
        sizes = {runner.pack(root, *cs, keep=False) or runner.vr.n_nodes for cs in cand_sets}
        if len(sizes) != 1:
            raise RuntimeError(f"candidate variants give different trie sizes {sorted(sizes)}")
        # eager warm-up (GEMM plans), then one graph for the device step
        runner.pack(root, *cand_sets[0], keep=False)
        runner.device_step(k_cache, v_cache, P)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            runner.device_step(k_cache, v_cache, P)
        stream.synchronize()
    setup_s = time.time() - t_setup
    calibration_copy(args.calibrate_copy_mib, dev)

    # per-phase breakdown on eager steps (outside the timed steps)
    with torch.cuda.stream(stream):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        cfg, vr = mcfg, runner.vr
        phase = {"projections_us": 0.0, "attention_us": 0.0, "other_us": 0.0}
        reps = 3
        for _ in range(reps):
            runner.pack(root, *cand_sets[0], keep=False)
            vr.upload_tree()
            N = vr.n_nodes
            ooo.embed_rows(runner.emb, vr.token, N, runner.h)
            ev[0].record(stream)
            ooo.rmsnorm(runner.h, runner.layers[0]["in_norm"], cfg.eps, runner.x, n_rows=N)
            ev[1].record(stream)
            stream.synchronize()
            phase["other_us"] += 1e3 * ev[0].elapsed_time(ev[1])
            for l, w in enumerate(runner.layers):
                # the runner's fused calls: projections include their fused
                # epilogues (norms, rotation and cache writes, residual adds)
                ev[0].record(stream)
                ooo.linear_qk_norm_rope(runner.x, w["w_qkv"], w["q_norm"], w["k_norm"], cfg.eps, vr.depth, N, P,
                                        cfg.rope_theta, cfg.n_q_heads, cfg.n_kv_heads, runner.q, k_cache[l],
                                        v_cache[l], runner.lin_ws)
                ev[1].record(stream)
                vr.attention(l, runner.q, k_cache[l], v_cache[l], P)
                ev[2].record(stream)
                o = vr.out[l].view(cfg.max_nodes, cfg.n_q_heads * cfg.head_dim)
                ooo.linear_add_rmsnorm(o, w["w_o"], runner.h, w["post_norm"], cfg.eps, runner.x, runner.lin_ws,
                                       n_rows=N)
                ooo.linear(runner.x, w["w_gu"], runner.act, ooo.EPI_SWIGLU_BF16, runner.lin_ws, n_rows=N)
                last = l + 1 == len(runner.layers)
                ooo.linear_add_rmsnorm(runner.act, w["w_down"], runner.h,
                                       runner.final_norm if last else runner.layers[l + 1]["in_norm"], cfg.eps,
                                       runner.xf if last else runner.x, runner.lin_ws, n_rows=N)
                ev[3].record(stream)
                stream.synchronize()
                phase["projections_us"] += 1e3 * (ev[0].elapsed_time(ev[1]) + ev[2].elapsed_time(ev[3]))
                phase["attention_us"] += 1e3 * ev[1].elapsed_time(ev[2])
        phase = {k: round(v / reps, 1) for k, v in phase.items()}

        Ls = []
        for i in range(args.warmup):
            runner.pack(root, *cand_sets[i % n_variants], keep=False)
            graph.replay()
            stream.synchronize()
            runner.result()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(args.steps):
            runner.pack(root, *cand_sets[i % n_variants], keep=False)
            graph.replay()
            stream.synchronize()
            Ls.append(runner.result().L)
        torch.cuda.synchronize()
        elapsed = time.perf_counter() - t0
    planted = [depths[i % n_variants] for i in range(args.steps)]
    if Ls != planted:
        print(f"note: {sum(a != b for a, b in zip(Ls, planted))} of {args.steps} steps accepted a different "
              f"length than planted", file=sys.stderr)
    w_bytes = mcfg.weight_bytes()
    proj_gbs = w_bytes / (phase["projections_us"] * 1e-6) / 1e9
    step_s = elapsed / args.steps
    out = {
        "metric": MODEL_METRIC,
        "value": round(args.steps / elapsed, 2),
        "unit": "verify steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(1e3 * step_s, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (random weights; each step's first candidate is the model's own greedy continuation)",
        "config": {"workload": f"{mcfg.name}: {mcfg.description}", "n_layers": mcfg.n_layers, "hidden": mcfg.hidden,
                   "q_heads": mcfg.n_q_heads, "kv_heads": mcfg.n_kv_heads, "head_dim": mcfg.head_dim,
                   "intermediate": mcfg.intermediate, "vocab": mcfg.vocab, "prefix_len": P,
                   "trie_nodes": int(runner.vr.n_nodes), "launch": "one hip-graph per step"},
        "tokens_per_s": round(float(np.sum(np.array(Ls) + 1)) / elapsed, 1),
        "mean_accepted_plus_bonus": round(float(np.mean(np.array(Ls) + 1)), 3),
        "phase_us_eager": phase,
        "roofline": {"bound": "hbm", "kernel": ("projections over all layers (qkv with norms/rotation, o_proj and down with residual add + "
                                "RMSNorm, gate+up with SwiGLU; streaming + epilogue kernels)"),
                     "achieved": round(proj_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(proj_gbs / HBM_PEAK_GBS, 4),
                     "traffic": recorded_traffic(mcfg.name, "projections"), "bytes_per_launch": w_bytes,
                     "us_per_launch": phase["projections_us"]},
        "step_weight_gbs": round(w_bytes / step_s / 1e9, 1),
        "setup_s": round(setup_s, 1),
    }
    if not args.no_cpu_baseline:
        del k_cache, v_cache, runner
        torch.cuda.empty_cache()
        out["cpu_baseline"] = model_cpu_baseline(mcfg, args.cpu_seconds)
    print(json.dumps(out), flush=True)


DECODE_METRIC = ("decode tokens/s (greedy, batch 1, asynchronous hint), Qwen3-8B decoder (36 layers, random "
                 "weights), 64-node tries, 4k prefix")
HIDDEN_PUSH = 12.0  # planted LM-head rows: N(0,1) noise plus this times the unit W row of the greedy token
DECODE_WORKLOADS = {"qwen3-8b-decode": "qwen3-8b-model", "small-decode": "small-model"}
DECODE_TOKENS = 256       # tokens generated per request
DECODE_HINT_DELAY_MS = 20  # the sidecar's hint arrives this long after the request starts
DECODE_HINT_ERROR_PERIOD = 24  # one wrong token in this many of the hint's


def bench_decode(args):
    """Whole requests of DECODE_TOKENS greedy tokens through ``DecodeLoop``:
    plain decoding (one token per verify step), the native candidates alone,
    and the native candidates plus a hint that a thread delivers
    DECODE_HINT_DELAY_MS after the request starts (Eq. 3: picked up at the
    first candidate boundary after it is ready).  Wall time per request
    includes the host's candidate construction, readiness checks, merging,
    packing and the per-round synchronisation."""
    import concurrent.futures
    import dataclasses

    import torch

    from paper_2608_00814_amd import model_workload as mw
    from paper_2608_00814_amd import ooo
    from paper_2608_00814_amd import workload as wl
    from paper_2608_00814_amd.decode import DecodeLoop, SidecarHint
    from paper_2608_00814_amd.model import ModelRunner

    ooo.lib()
    base = mw.MODEL_CONFIGS[DECODE_WORKLOADS[args.workload]]
    G = DECODE_TOKENS
    mcfg = dataclasses.replace(base, cap=base.prefix_len + G + 2 * base.max_nodes)
    dev = torch.device("cuda:0")
    P0 = mcfg.prefix_len
    seed = 0
    t_setup = time.time()
    # Synthetic weights of the decoder's shapes whose greedy continuation has
    # wide logit margins: embeddings times 16 (exact in bf16) dominate the
    # residual stream, and LM-head row v is the embedding row of perm^-1(v),
    # so the greedy next token of t is perm(t).  (With plain random weights
    # the top two logits nearly tie at many positions, and rounding that
    # differs between trie shapes flips them, so no hint prepared in advance
    # would stay aligned.)  The kernels' work is the same either way.
    emb = wl.to_bf16_bits(wl.bf16_to_f32(mw.embedding(mcfg, seed)) * np.float32(16.0))
    perm = np.random.default_rng(7).permutation(mcfg.vocab)
    lm = np.empty_like(emb)
    lm[perm] = emb
    layers = (mw.layer_weights(mcfg, seed, l) for l in range(mcfg.n_layers))
    runner = ModelRunner(mcfg, layers, emb, mw.final_norm(mcfg, seed), lm, dev)
    del emb, lm
    shp = (mcfg.n_layers, mcfg.n_kv_heads, mcfg.cap, mcfg.head_dim)
    k_cache = torch.zeros(shp, dtype=torch.bfloat16, device=dev)
    v_cache = torch.zeros(shp, dtype=torch.bfloat16, device=dev)
    for l in range(mcfg.n_layers):
        k, v = mw.prefix_kv(mcfg, seed, l)
        k_cache[l].copy_(torch.from_numpy(k.view(np.int16)).view(torch.bfloat16))
        v_cache[l].copy_(torch.from_numpy(v.view(np.int16)).view(torch.bfloat16))
    torch.cuda.synchronize()
    pcfg = wl.CONFIGS["qwen3-8b"]
    eos = mcfg.vocab - 1
    root = wl.candidates_for(pcfg, seed, 0).root_token % eos
    stream = torch.cuda.Stream()

    def native_lanes(r, y):
        # stand-ins for the schema chain and two retrieved calls (the path
        # workload's non-hint lanes of round r); they are rarely right here
        return [[t % eos for t in q] for q in wl.candidates_for(pcfg, seed, r).seqs[1:]]

    def no_lanes(r, y):
        return []

    loops = {}

    def request(kind, views=None):
        """One request; returns (seconds, records, loop)."""
        hint = None
        ex = None
        native = no_lanes if kind == "plain" else native_lanes
        # one loop object per kind keeps its captured graphs across requests
        loop = loops.get(kind)
        if loop is None:
            loop = DecodeLoop(runner, k_cache, v_cache, P0, root, native, n_lanes=8, graphs=not args.no_graph,
                              stream=stream)
            loops[kind] = loop
        loop.P, loop.committed, loop.rounds = P0, [root], 0
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        if views is not None:
            ex = concurrent.futures.ThreadPoolExecutor(max_workers=1)
            fut = ex.submit(lambda: (time.sleep(DECODE_HINT_DELAY_MS / 1e3), views)[1])
            loop.hint = SidecarHint(fut, eos)
        else:
            loop.hint = None
        recs = loop.run(max_rounds=G, max_new_tokens=G)
        el = time.perf_counter() - t0
        if ex is not None:
            ex.shutdown(wait=True)
        return el, recs, loop

    # The hint's content: the model's own output as the tree-verifying loop
    # produces it (plain one-token steps round differently and can part from
    # it at a near tie of the random model), found as the fixed point of
    # hinted runs, then corrupted at every DECODE_HINT_ERROR_PERIOD-th token
    # (an imperfect sidecar: each error costs a rejection and a re-alignment
    # of the suffix match at a later round, Section 4.4).
    _, recs, loop = request("plain")
    greedy = loop.committed[1:G + 1]
    rs = np.random.default_rng(3)
    decoys = [[int(t) for t in rs.integers(0, eos, size=200)] for _ in range(3)]
    target = greedy
    for _ in range(3):
        _, _, lp = request("hint", decoys + [[root] + target])
        out = lp.committed[1:G + 1]
        if out == target:
            break
        target = out
    noisy = list(target)
    for i in range(DECODE_HINT_ERROR_PERIOD - 1, len(noisy), DECODE_HINT_ERROR_PERIOD):
        noisy[i] = (noisy[i] + 1) % eos
    views = decoys + [[root] + noisy]
    setup_s = time.time() - t_setup
    results = {}
    for kind, vw in (("plain", None), ("native", None), ("hint", views)):
        for _ in range(max(1, args.warmup)):
            request(kind, vw)  # captures the graphs of the trie sizes this kind produces
        n_graphs = len(loops[kind]._graphs)
        times, toks, rounds, first, agree, agree_t = [], [], [], [], [], []
        for _ in range(args.steps):
            el, recs, lp = request(kind, vw)
            got = lp.committed[1:G + 1]
            # tree steps round differently from one-token steps (other GEMM
            # row tilings), so at a near tie of the random model the two may
            # part; report how far they agree
            n_same = next((i for i, (x, y) in enumerate(zip(got, greedy)) if x != y), min(len(got), len(greedy)))
            agree.append(n_same)
            agree_t.append(next((i for i, (x, y) in enumerate(zip(got, target)) if x != y),
                                min(len(got), len(target))))
            times.append(el)
            toks.append(sum(len(r.committed) for r in recs))
            rounds.append(len(recs))
            if lp.hint is not None:
                first.append(lp.hint.first_ready_round)
        results[kind] = {"s_per_request": float(np.median(times)), "tokens": int(np.median(toks)),
                         "rounds": int(np.median(rounds)), "captures_in_timed": len(loops[kind]._graphs) - n_graphs,
                         "tokens_agreeing_with_plain": int(min(agree)),
                         "tokens_agreeing_with_hint_target": int(min(agree_t)),
                         "hint_first_round": first,
                         "host_us_per_round": round(float(np.mean([r.host_us for r in recs])), 1),
                         "device_us_per_round": round(float(np.mean([r.device_us for r in recs])), 1)}
    h = results["hint"]
    tps = {k: v["tokens"] / v["s_per_request"] for k, v in results.items()}
    out = {
        "metric": DECODE_METRIC,
        "value": round(tps["hint"], 1),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(1e3 * h["s_per_request"], 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": ("synthetic (random layer weights, embeddings x16 and LM-head rows = permuted embedding rows; after "
                 f"decoy views the hint holds the model's own output with every {DECODE_HINT_ERROR_PERIOD}th token "
                 "wrong)"),
        "config": {"workload": f"{args.workload}: {G}-token requests, {mcfg.description}", "n_layers": mcfg.n_layers,
                   "hidden": mcfg.hidden, "vocab": mcfg.vocab, "prefix_len": P0, "max_nodes": mcfg.max_nodes,
                   "max_depth": mcfg.max_depth, "hint_delay_ms": DECODE_HINT_DELAY_MS,
                   "hint_error_period": DECODE_HINT_ERROR_PERIOD,
                   "launch": "eager" if args.no_graph else "one hip-graph per trie size, prefix from device memory"},
        "step": "one request of %d tokens" % G,
        "tokens_per_s": {k: round(v, 1) for k, v in tps.items()},
        "speedup_vs_plain": {k: round(tps[k] / tps["plain"], 3) for k in tps},
        "per_kind": results,
        "roofline": None,
        "setup_s": round(setup_s, 1),
    }
    if not args.no_cpu_baseline:
        del k_cache, v_cache, runner, loops
        torch.cuda.empty_cache()
        cb = model_cpu_baseline(mcfg, args.cpu_seconds)
        per_round = h["tokens"] / max(1, h["rounds"])
        out["cpu_baseline"] = {"value": cb["value"] * per_round, "unit": "tokens/s", "cores": cb["cores"],
                               "kind": "oracle", "sample": cb["sample"] + f"; times {per_round:.2f} tokens per "
                               "round of the hint run"}
    print(json.dumps(out), flush=True)


LOOP_METRIC = "decode verify steps/s over consecutive steps with compaction (wall clock, per-step host sync)"


def bench_path_loop(args):
    """Consecutive verify steps of the path with compaction, each step's root
    the previous step's bonus token and the prefix growing by L + 1, timed by
    the wall clock over all steps including the per-step synchronisation.
    One captured graph per trie size, replayed with the prefix length read
    from device memory.  Per step the host builds the step's candidates with
    the workload generator (a stand-in for the schema chain, retrieved calls
    and, from step 30 on, the hint), packs them and stages the planted
    LM-head rows; the node queries and K/V rows are not restaged (their
    values do not change the work)."""
    import torch

    from paper_2608_00814_amd import ooo
    from paper_2608_00814_amd import workload as wl
    from paper_2608_00814_amd.step import VerifyRunner

    ooo.lib()
    cfg = wl.CONFIGS[args.workload]
    steps = args.steps if args.steps > 0 else cfg.steps
    dev = torch.device("cuda:0")
    seed = 0
    t_setup = time.time()
    bound = cfg.cap - cfg.max_nodes
    runner = VerifyRunner(cfg.n_layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden, cfg.vocab,
                          cfg.max_nodes, cfg.max_depth, torch.bfloat16, dev, max_prefix=bound)
    w = wl.lm_head_weight(cfg, seed)
    w_rows = torch.from_numpy(np.ascontiguousarray(w).view(np.int16)).view(torch.bfloat16).to(dev)
    del w
    runner.set_weight(w_rows.clone())
    inv_norm = torch.rsqrt((w_rows.float() ** 2).sum(1))  # staging: X rows pushed along W[tau] / |W[tau]|
    g = torch.Generator(device=dev).manual_seed(seed)
    z = torch.randn(cfg.max_nodes, cfg.hidden, device=dev, generator=g)
    x_buf = torch.empty(cfg.max_nodes, cfg.hidden, dtype=torch.bfloat16, device=dev)
    shp = (cfg.n_layers, cfg.n_kv_heads, cfg.cap, cfg.head_dim)
    k_cache = torch.randn(shp, device=dev, generator=g).to(torch.bfloat16)
    v_cache = torch.randn(shp, device=dev, generator=g).to(torch.bfloat16)
    q_layers = [torch.randn(cfg.max_nodes, cfg.n_q_heads, cfg.head_dim, device=dev, generator=g).to(torch.bfloat16)
                for _ in range(cfg.n_layers)]
    for n in range(1, cfg.max_nodes + 1):
        runner.ensure_workspace(bound, n)
    ws_ptr = runner.attn_ws.data_ptr()
    torch.cuda.synchronize()
    setup_s = time.time() - t_setup
    stream = torch.cuda.Stream()
    graphs = {}
    done = torch.cuda.Event()

    def run(n_steps):
        root = wl.candidates_for(cfg, seed, 0).root_token
        P = cfg.prefix_len
        gen_s = dev_s = 0.0
        Ls, mismatch, captures = [], 0, 0
        for s_ in range(n_steps):
            t0 = time.perf_counter()
            cands = wl.candidates_for(cfg, seed, s_, root_token=root)
            packed = runner.pack(root, *cands.csr())
            tau, d = wl.designated_tokens(cfg, seed, s_, cands, packed["token"], packed["parent"])
            t1 = time.perf_counter()
            N = packed["n_nodes"]
            with torch.cuda.stream(stream):
                tdev = torch.from_numpy(tau.astype(np.int64)).to(dev, non_blocking=False)
                x_buf[:N].copy_(z[:N] + HIDDEN_PUSH * w_rows[tdev].float() * inv_norm[tdev][:, None])
                runner.set_prefix(P)
                gr = graphs.get(N)
                if gr is None:
                    if runner.attn_ws.data_ptr() != ws_ptr:
                        raise RuntimeError("attention workspace moved after a capture")
                    gr = torch.cuda.CUDAGraph()
                    with torch.cuda.graph(gr, stream=stream):
                        runner.device_step(q_layers, k_cache, v_cache, x_buf, bound, prefix_dev=runner.prefix_dev)
                    graphs[N] = gr
                    captures += 1
                gr.replay()
                done.record(stream)
            done.synchronize()
            res = runner.result()
            t2 = time.perf_counter()
            gen_s += t1 - t0
            dev_s += t2 - t1
            mismatch += res.L != d
            Ls.append(res.L)
            root = res.bonus
            P += res.L + 1
            if P > bound:
                break
        return {"Ls": Ls, "gen_s": gen_s, "dev_s": dev_s, "mismatch": mismatch, "captures": captures, "P": P}

    run(min(steps, max(args.warmup, 35)))  # captures the graphs of the trie sizes the steps produce
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r = run(steps)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    n_done = len(r["Ls"])
    committed = int(np.sum(np.array(r["Ls"]) + 1))
    out = {
        "metric": LOOP_METRIC,
        "value": round(n_done / elapsed, 2),
        "unit": "verify steps/s",
        "n_gpus": 1,
        "steps": n_done,
        "warmup": max(args.warmup, 35),
        "ms_per_step": round(1e3 * elapsed / n_done, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (generator candidates per step, planted acceptance)",
        "config": {"workload": f"{cfg.name}: {cfg.description}", "n_layers": cfg.n_layers, "q_heads": cfg.n_q_heads,
                   "kv_heads": cfg.n_kv_heads, "head_dim": cfg.head_dim, "prefix_len": cfg.prefix_len,
                   "final_prefix_len": r["P"], "trie_nodes": cfg.max_nodes, "hidden": cfg.hidden,
                   "vocab": cfg.vocab, "launch": "one hip-graph per trie size, prefix from device memory"},
        "tokens_per_s": round(committed / elapsed, 1),
        "mean_accepted_plus_bonus": round(committed / n_done, 3),
        "generator_ms_per_step": round(1e3 * r["gen_s"] / n_done, 3),
        "staging_and_device_ms_per_step": round(1e3 * r["dev_s"] / n_done, 3),
        "steps_accepting_other_than_planted": r["mismatch"],
        "graph_captures_in_timed_steps": r["captures"],
        "roofline": None,
        "setup_s": round(setup_s, 1),
    }
    if not args.no_cpu_baseline:
        del k_cache, v_cache, q_layers, runner, graphs
        torch.cuda.empty_cache()
        cb = cpu_baseline(cfg, args.cpu_seconds)
        out["cpu_baseline"] = cb
    print(json.dumps(out), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="qwen3-8b")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-graph", action="store_true", help="launch every kernel eagerly")
    ap.add_argument("--no-others", action="store_true",
                    help="skip the kernel timings at the other workloads' shapes (default run only)")
    ap.add_argument("--loop", action="store_true",
                    help="consecutive verify steps with compaction from the workload's prefix (wall clock)")
    ap.add_argument("--record-traffic", nargs=2, metavar=("FETCH_CSV", "WRITE_CSV"),
                    help="write profiles/hbm_traffic_<workload>.json from the counter_collection.csv files of a "
                         "FETCH_SIZE and a WRITE_SIZE rocprofv3 run (no GPU needed)")
    ap.add_argument("--calibrate-copy-mib", type=int, default=0,
                    help="one plain copy of this many MiB after setup (byte-counter calibration)")
    args = ap.parse_args()
    if args.record_traffic:
        rec = traffic_record(args.workload, *args.record_traffic, calibrate_mib=args.calibrate_copy_mib or 1024)
        path = os.path.join(ROOT, "profiles", f"hbm_traffic_{args.workload}.json")
        with open(path, "w") as f:
            json.dump(rec, f, indent=1)
        print(json.dumps({k: v["bytes_per_launch"] for k, v in rec.items() if isinstance(v, dict)}))
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (asked for {args.gpus}); the path runs on a single MI355X.",
              file=sys.stderr)
        sys.exit(2)

    from paper_2608_00814_amd import model_workload as mw
    if args.workload in mw.MODEL_CONFIGS:
        bench_model(args)
        return
    if args.workload in DECODE_WORKLOADS:
        bench_decode(args)
        return
    if args.loop:
        bench_path_loop(args)
        return

    import torch

    from paper_2608_00814_amd import ooo
    from paper_2608_00814_amd import workload as wl
    from paper_2608_00814_amd.step import VerifyRunner

    if not torch.cuda.is_available():
        print("bench.py needs a ROCm GPU", file=sys.stderr)
        sys.exit(1)
    ooo.lib()  # fail loudly if the native library is missing
    cfg = wl.CONFIGS[args.workload]
    dev = torch.device("cuda:0")
    tdt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    P = cfg.prefix_len
    t_setup = time.time()

    def up(a):
        if cfg.dtype == "bf16":
            return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(dev)
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev)

    # --- resident inputs ---------------------------------------------------
    n_variants = 4  # distinct candidate sets, cycled over the timed steps
    cand_sets = [wl.candidates_for(cfg, s, 0) for s in range(n_variants)]
    runner = VerifyRunner(cfg.n_layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.hidden, cfg.vocab,
                          cfg.max_nodes, cfg.max_depth, tdt, dev, max_prefix=P)
    csr = [c.csr() for c in cand_sets]
    packs = [runner.pack(c.root_token, *x) for c, x in zip(cand_sets, csr)]
    N = packs[0]["n_nodes"]
    assert all(p["n_nodes"] == N for p in packs)
    w = wl.lm_head_weight(cfg, 0)
    w_dev = up(w)
    runner.set_weight(w_dev)  # packed once for streaming; not part of a step
    del w_dev
    hid = []
    for s, (c, p) in enumerate(zip(cand_sets, packs)):
        tau, _ = wl.designated_tokens(cfg, s, 0, c, p["token"], p["parent"])
        hid.append(up(wl.hidden_rows(cfg, s, 0, w, tau, N)))
    del w
    shp = (cfg.n_layers, cfg.n_kv_heads, cfg.cap, cfg.head_dim)
    k_cache = torch.zeros(shp, dtype=tdt, device=dev)
    v_cache = torch.zeros(shp, dtype=tdt, device=dev)
    q_layers = []
    for l in range(cfg.n_layers):
        kc, vc = wl.layer_cache(cfg, 0, l, N)
        k_cache[l].copy_(up(kc))
        v_cache[l].copy_(up(vc))
        q_layers.append(up(wl.queries(cfg, 0, 0, l, N)))
    runner.ensure_workspace(P)
    torch.cuda.synchronize()
    setup_s = time.time() - t_setup

    calibration_copy(args.calibrate_copy_mib, dev)

    stream = torch.cuda.Stream()  # default priority
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]

    def attend():
        for l in range(cfg.n_layers):
            runner.attention(l, q_layers[l], k_cache[l], v_cache[l], P)

    def tail():
        runner.accept()
        runner.compact(k_cache, v_cache, P)
        runner.download()

    graphs = None
    with torch.cuda.stream(stream):
        runner.pack(cand_sets[0].root_token, *csr[0])
        if not args.no_graph:
            # eager warm-up of every kernel before capture
            runner.upload_tree()
            attend()
            runner.lm_head(hid[0])
            tail()
            stream.synchronize()
            ga, gt = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
            with torch.cuda.graph(ga, stream=stream):
                attend()
            with torch.cuda.graph(gt, stream=stream):
                tail()
            graphs = (ga, gt)
        stream.synchronize()

        lm_ms, attn_ms, Ls = [], [], []

        def one_step(i, timed):
            v = i % n_variants
            runner.pack(cand_sets[v].root_token, *csr[v], keep=False)
            runner.upload_tree()
            ev[0].record(stream)
            if graphs:
                graphs[0].replay()
            else:
                attend()
            ev[1].record(stream)
            runner.lm_head(hid[v])
            ev[2].record(stream)
            if graphs:
                graphs[1].replay()
            else:
                tail()
            stream.synchronize()
            r = runner.result()
            if timed:
                Ls.append(r.L)
                attn_ms.append(ev[0].elapsed_time(ev[1]))
                lm_ms.append(ev[1].elapsed_time(ev[2]))
            return r

        for i in range(args.warmup):
            one_step(i, False)
        torch.cuda.synchronize()
        step_s = []
        t0 = time.perf_counter()
        for i in range(args.steps):
            ts = time.perf_counter()
            one_step(i, True)
            step_s.append(time.perf_counter() - ts)
        torch.cuda.synchronize()
        elapsed = time.perf_counter() - t0

        # A working set that fits the 256 MiB last-level cache (MALL) of the
        # GPU is timed once more with a 512 MiB buffer written before every
        # step, outside the attention and LM-head brackets, so that their
        # inputs come from HBM.
        work_set = cfg.n_layers * attention_bytes(cfg, N) + lmhead_bytes(cfg, N)
        flushed = None
        if work_set <= (512 << 20):
            flush = torch.empty(512 << 18, dtype=torch.float32, device=dev)
            kept = (attn_ms, lm_ms, Ls)
            attn_ms, lm_ms, Ls = [], [], []
            for i in range(args.steps):
                flush.fill_(float(i))
                one_step(i, True)
            flushed = (attn_ms, lm_ms)
            attn_ms, lm_ms, Ls = kept
            del flush

    ms_per_step = 1e3 * elapsed / args.steps
    steps_per_s = args.steps / elapsed
    tokens_per_s = float(np.sum(np.array(Ls) + 1)) / elapsed
    lm_us = 1e3 * float(np.mean(lm_ms))
    attn_us = 1e3 * float(np.mean(attn_ms))
    hint_us, hint_tokens = time_hint_merge(cfg, cand_sets)
    attn_call_us = attn_us / cfg.n_layers
    a_bytes = attention_bytes(cfg, N)
    a_gbs = a_bytes / (attn_call_us * 1e-6) / 1e9
    lm_b = lmhead_bytes(cfg, N)
    lm_gbs = lm_b / (lm_us * 1e-6) / 1e9
    path_gbs = (cfg.n_layers * a_bytes + lm_b) / ((attn_us + lm_us) * 1e-6) / 1e9
    # attention flops over the prefix keys (4 Hq N P D: scores and P V)
    a_flops = 4.0 * cfg.n_q_heads * N * P * cfg.head_dim
    a_tflops = a_flops / (attn_call_us * 1e-6) / 1e12
    mfma_peak = MFMA_PEAK_TFLOPS if cfg.dtype == "bf16" else FP32_PEAK_TFLOPS
    mfma_bound = a_flops / a_bytes > mfma_peak * 1e12 / (HBM_PEAK_GBS * 1e9)

    copy_gbs = copy_bandwidth_gbs(dev)
    cpu_model, cpu_cores = host_cpu()
    st_stats = step_time_stats(step_s)
    out = {
        "metric": METRIC,
        "value": round(steps_per_s, 2),
        "unit": "verify steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": cfg.dtype,
        "data": "synthetic",
        "config": {"workload": f"{cfg.name}: {cfg.description}", "n_layers": cfg.n_layers,
                   "q_heads": cfg.n_q_heads, "kv_heads": cfg.n_kv_heads, "head_dim": cfg.head_dim,
                   "prefix_len": P, "trie_nodes": N, "hidden": cfg.hidden, "vocab": cfg.vocab,
                   "launch": "eager" if args.no_graph else "hip-graph per phase, LM head eager"},
        "tokens_per_s": round(tokens_per_s, 1),
        "hint_merge_us": round(hint_us, 2),
        "hint_bank_tokens": hint_tokens,
        "mean_accepted_plus_bonus": round(float(np.mean(np.array(Ls) + 1)), 3),
        "attention_us_per_step": round(attn_us, 2),
        "attention_us_per_layer": round(attn_call_us, 3),
        "lmhead_us": round(lm_us, 2),
        "path_hbm_gbs": round(path_gbs, 1),
        "path_hbm_frac": round(path_gbs / HBM_PEAK_GBS, 4),
        "roofline": ({"bound": "mfma", "kernel": "ooo_tree_attn (tree_attn_bf16_kernel + tree_attn_combine_kernel)",
                      "achieved": round(a_tflops, 1), "peak": mfma_peak, "unit": "TFLOP/s",
                      "frac": round(a_tflops / mfma_peak, 4), "traffic": recorded_traffic(cfg.name, "ooo_tree_attn"),
                      "flops_per_launch": a_flops, "bytes_per_launch": a_bytes,
                      "us_per_launch": round(attn_call_us, 3)} if mfma_bound else
                     {"bound": "hbm", "kernel": "ooo_tree_attn (tree_attn_bf16_kernel + tree_attn_combine_kernel)",
                      "achieved": round(a_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                      "frac": round(a_gbs / HBM_PEAK_GBS, 4), "traffic": recorded_traffic(cfg.name, "ooo_tree_attn"),
                      "bytes_per_launch": a_bytes,
                      "us_per_launch": round(attn_call_us, 3)}),
        "attention_hbm_frac": round(a_gbs / HBM_PEAK_GBS, 4),
        "attention_mfma_frac": round(a_tflops / mfma_peak, 4),
        "roofline_lmhead": {"bound": "hbm", "kernel": "ooo_lmhead_argmax (lmhead_bf16_kernel + lmhead_finalize_kernel)",
                            "achieved": round(lm_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                            "frac": round(lm_gbs / HBM_PEAK_GBS, 4),
                            "traffic": recorded_traffic(cfg.name, "ooo_lmhead_argmax"), "bytes_per_launch": lm_b,
                            "us_per_launch": round(lm_us, 2)},
        "step_time": st_stats,
        "steps_per_s_at_median": round(1e3 / st_stats["median_ms"], 2),
        "tokens_per_s_at_paper_mat": tokens_at_mat(steps_per_s),
        "copy_gbs": round(copy_gbs, 1),
        "path_frac_of_copy": round(path_gbs / copy_gbs, 4),
        "attention_frac_of_copy": round(a_gbs / copy_gbs, 4),
        "host": {"cpu_model": cpu_model, "cores": cpu_cores},
        "paper_context": PAPER_CONTEXT,
        "setup_s": round(setup_s, 1),
    }
    if flushed is not None:
        f_attn_us = 1e3 * float(np.mean(flushed[0]))
        f_lm_us = 1e3 * float(np.mean(flushed[1]))
        f_path_gbs = (cfg.n_layers * a_bytes + lm_b) / ((f_attn_us + f_lm_us) * 1e-6) / 1e9
        out["mall_flushed"] = {"note": "512 MiB written before every step (the working set fits the 256 MiB MALL)",
                               "attention_us_per_layer": round(f_attn_us / cfg.n_layers, 3),
                               "lmhead_us": round(f_lm_us, 2), "path_hbm_gbs": round(f_path_gbs, 1),
                               "path_hbm_frac": round(f_path_gbs / HBM_PEAK_GBS, 4)}
    del k_cache, v_cache
    torch.cuda.empty_cache()
    if args.workload == "qwen3-8b" and not args.no_others and not args.no_graph:
        out["other_workloads"] = {name: secondary_rates(name, dev) for name in SECONDARY_WORKLOADS}
        shard = secondary_rates(tp8_shard_config(), dev)
        shard["note"] = ("one GPU's share of the Qwen3-8B step under 8-way tensor parallelism (1 KV head, "
                         "4 query heads, 1/8 of the vocabulary rows); the all-gather of N x 8 B per step "
                         "is not included")
        out["tp8_shard"] = shard
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg, args.cpu_seconds)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
