#!/usr/bin/env python3
"""Benchmark of the cluster-shared prefill-attention hot path on one MI355X.

One step = one pass of the whole path over one batch (SubGCache Sec. 3.4, cluster-wise): for
every cluster allocate its cache pages and prefill its prefix (K/V ingest + the prefix's causal
attention), map the batch's queries to clusters (host) and upload the plan, run the batched
suffix prefill of every query, release the pages.  All tensors are resident in HBM before the
timed region.  Prints ONE JSON line.
"""
from __future__ import annotations

import argparse
import contextlib
import gc
import json
import os
import sys
import time

import numpy as np


@contextlib.contextmanager
def no_gc():
    """Python's cyclic garbage collector off for a timed region, as in timeit: a full collection over the workload's
    objects takes 35 ms of host time (seventy steps of the headline configuration) and says nothing about the path.
    (Callers collect once before their untimed phase, so that the pause does not fall between it and the timed one.)"""
    gc.disable()
    try:
        yield
    finally:
        gc.enable()

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_TFLOPS = {"bf16": 2500.0, "fp8": 5000.0, "f32": 157.3}      # MI355X dense MFMA bf16 (= fp16) and fp8; fp32 (the same for matrix cores and vector)
HBM_PEAK_GBS = 8000.0

# HBM bytes per launch of the suffix attention kernel from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this
# file (not of the run that prints them: counters need the profiler), each counter scaled by what it reads for a
# plain copy of known size (--copy-calibration).  Keyed by workload; the runs and the arithmetic are written down
# in the named file under profiles/.  A workload that has not been measured this way reports null.
PROFILED_HBM_BYTES_PER_LAUNCH = {
    ("llama3_8b_layer", "16bit"): (3.126e8, "profiles/attn_mfma_suffix_llama3_8b_layer.md"),
    ("llama2_7b_ragged", "16bit"): (2.851e9, "profiles/suffix_prefill_all_configs.md"),
    ("llama3_8b_stack32", "16bit"): (9.791e8, "profiles/suffix_prefill_all_configs.md"),
    ("tiny_f32_mha", "16bit"): (1.041e7, "profiles/suffix_prefill_all_configs.md"),        # (the generic kernel, fp32 operands)
    ("llama70b_fp8_long", "fp8_first_product"): (2.078e10, "profiles/suffix_prefill_all_configs.md"),
}
# The same for one decode step of configs[1] (cached-prompt part 58.5 MB + own-keys kernel 95.9 MB) and for the QKV
# projection of its batch at d_model 4096.
PROFILED_DECODE_STEP_BYTES = {"llama3_8b_layer": (1.544e8, "profiles/decode_llama3_8b_layer.md")}
PROFILED_QKV_GEMM_BYTES = {("llama3_8b_layer", 4096): (1.583e9, "profiles/proj_gemm_llama3_8b_layer.md")}
TOLERANCE = {"f32": 2e-5, "bf16": 2e-2, "fp8_e4m3": 6e-2}     # max-abs bars against the fp64 oracle

# Other ceilings of the matrix-core attention kernel, beside the datasheet MFMA peak (all in TFLOP/s of attention flop):
# * per score (4 d = 512 flop at d = 128) the softmax needs one exp2 (two issue slots of 4 cycles per 64 lanes), half
#   a conversion and half a dot2 (one slot each): 3 slots x 4 cycles / 64 lanes = 0.1875 SIMD cycles, against
#   512 / 1024 = 0.5 SIMD cycles of matrix-core time: the vector unit alone would carry 2500 x 0.5 / 0.1875;
# * if the two did not overlap at all (one issue port, one wavefront): 2500 x 0.5 / 0.6875;
# * what a kernel of nothing but MFMA instructions sustains on unit-scale random operands (the chip lowers its clock
#   under the data-dependent power): 1680 (binary16) and 1820 (bf16), 1750 for this kernel's half-and-half mix
#   (measured: profiles/gfx950_microbenchmarks.md).
CO_LIMITS_TFLOPS = {"valu_softmax": 2500.0 * 0.5 / 0.1875, "mfma_and_valu_not_overlapped": 2500.0 * 0.5 / 0.6875,
                    "mfma_sustained_on_random_operands": 1750.0}


def co_limits(achieved_tflops: float) -> dict:
    return {k: {"peak": v, "frac": achieved_tflops / v} for k, v in CO_LIMITS_TFLOPS.items()}


def copy_calibration() -> int:
    """A plain device copy of known size, for scaling the profiler's FETCH_SIZE / WRITE_SIZE counters."""
    import torch
    n = 256 << 20
    src = torch.empty(n, dtype=torch.uint8, device="cuda:0").fill_(1)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    for _ in range(10):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": n, "copy_bytes_written": n, "copies": 10}), flush=True)
    return 0



def prefix_flops(w) -> float:
    P = w.prefix_len.astype(np.float64)
    return float(4.0 * w.n_q_heads * w.head_dim * np.sum(P * (P + 1.0) / 2.0))


def oracle_on_queries(w, queries, layer=0, caches=None):
    """The fp64 oracle on the given queries of a workload: (seconds, flop, o [rows][Hq][d], packed row indices)."""
    from oracle import oracle as orc
    caches = {} if caches is None else caches
    qs, ks, vs, cu, rows = [], [], [], [0], []
    wcu = w.cu_seqlens
    for n in queries:
        c = int(w.labels[n])
        if c not in caches:
            k, v = w.prefix_kv(c, layer)
            ck, cv, _, _ = orc.prefix_prefill(None, k, v, w.rope_base)
            if w.kv_dtype == "fp8_e4m3":
                ck, cv = orc.quantise_e4m3(ck)[2], orc.quantise_e4m3(cv)[2]
            caches[c] = (ck, cv)
        q, k, v = w.suffix_qkv_query(n, layer)
        qs.append(q), ks.append(k), vs.append(v)
        cu.append(cu[-1] + q.shape[0])
        rows.extend(range(int(wcu[n]), int(wcu[n + 1])))
    empty = np.zeros((0, w.n_kv_heads, w.head_dim))
    cks = [caches[c][0] if c in caches else empty for c in range(w.n_clusters)]
    cvs = [caches[c][1] if c in caches else empty for c in range(w.n_clusters)]
    q, k, v = (np.concatenate(x).astype(np.float64) for x in (qs, ks, vs))
    labels = w.labels[list(queries)]
    t0 = time.perf_counter()
    o, _ = orc.suffix_prefill_batched(labels, np.array(cu), cks, cvs, q, k, v, w.rope_base)
    dt = time.perf_counter() - t0
    S = w.suffix_len[list(queries)].astype(np.float64)
    P = w.prefix_len[labels].astype(np.float64)
    fl = float(4.0 * w.n_q_heads * w.head_dim * np.sum(S * (P + (S + 1) / 2)))
    return dt, fl, o, np.array(rows, dtype=np.int64)


def error_against_oracle(o_gpu_rows: np.ndarray, o_ref: np.ndarray, kv_dtype: str, what: str):
    """max-abs and relative error of GPU rows against the oracle's (outside any timed region)."""
    d = np.abs(o_gpu_rows.astype(np.float64) - o_ref)
    rms = float(np.sqrt(np.mean(o_ref ** 2))) if o_ref.size else 0.0
    mx = float(d.max()) if d.size else 0.0
    return {"max_abs_err": mx, "rel_err": mx / rms if rms > 0 else 0.0, "rms_ref": rms, "bar": TOLERANCE[kv_dtype],
            "within_bar": bool(mx <= TOLERANCE[kv_dtype]), "rows_checked": int(o_ref.shape[0]), "checked": what}


def cpu_baseline(w, budget_s: float):
    """Times the fp64 oracle, as it stands, on a bounded sample of the same workload's queries.  Returns the
    report, and the sample's packed row indices and oracle outputs for the error figures."""
    from oracle import oracle as orc
    rng = np.random.default_rng(0)
    picks = [int(n) for n in rng.permutation(w.n_queries) if w.suffix_len[n] > 0]
    caches = {}
    threads = orc.n_threads()
    probe = picks[:max(threads, 4)]
    dt, fl, _, _ = oracle_on_queries(w, probe, caches=caches)
    rate = fl / max(dt, 1e-6)
    per_query = fl / len(probe)
    n = int(min(len(picks), max(len(probe), budget_s * rate / per_query)))
    sample = picks[:n]
    dt, fl, o_ref, rows = oracle_on_queries(w, sample, caches=caches)
    rep = {"value": fl / dt / 1e12, "unit": "TFLOP/s", "cores": threads, "kind": "oracle",
           "sample": f"{len(sample)} of {w.n_queries} queries (all heads, all rows), {fl:.3e} flop in {dt:.2f} s",
           "us_per_query": dt / len(sample) * 1e6}
    return rep, rows, o_ref


def oracle_one_thread(index: int):
    """The oracle on every query of a (small) configuration with one OpenMP thread, in a child process of its own
    (the thread count is read when the library starts; the child never touches the GPU)."""
    import subprocess
    code = ("import json, sys; sys.path.insert(0, %r); import bench; from paper_2505_10951_amd import workloads; "
            "w = workloads.config(%d); dt, fl, _, _ = bench.oracle_on_queries(w, [n for n in range(w.n_queries) if w.suffix_len[n] > 0]); "
            "print(json.dumps({'value': fl / dt / 1e12, 'unit': 'TFLOP/s', 'cores': 1, 'kind': 'oracle', "
            "'sample': 'all %%d queries, %%.3e flop in %%.3f s' %% (w.n_queries, fl, dt), 'us_per_query': dt / w.n_queries * 1e6}))") % (ROOT, index)
    env = dict(os.environ, OMP_NUM_THREADS="1")
    try:
        r = subprocess.run([sys.executable, "-c", code], env=env, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
        return json.loads(r.stdout.strip().splitlines()[-1])
    except Exception as e:                      # reported, never fatal: the figure is context
        return {"error": repr(e)}


def decode_measurement(s, w, layer, n_steps, dq, dk, dv, do, all_clusters, pq_ptrs, pk_ptrs, pv_ptrs, po_ptrs, stream):
    """Batched decode after the suffix prefill (the paper caps generation at 32 tokens): per-step time, HIP events
    around each step on the launch stream.  HBM-bound: every step has to read the cached K/V of each cluster
    once and every query's own keys once."""
    import torch
    from paper_2505_10951_amd import sgc
    from paper_2505_10951_amd.harness import to_device
    if s.plan is None or sgc.sgc_cache_free_pages(s.cache) == sgc.sgc_cache_total_pages(s.cache):
        for c in all_clusters:
            sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(w.prefix_len[c]))
        sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, all_clusters, layer, pq_ptrs, pk_ptrs, pv_ptrs, po_ptrs, None, stream)
    s.assign(w.labels, w.suffix_len)
    sgc.sgc_plan_enable_decode(s.ctx, s.plan, n_steps)
    sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, layer, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), do.data_ptr(),
                                   None, stream)
    tq, tk, tv = (to_device(x, w.io_dtype) for x in w.decode_qkv(0, layer))
    to = torch.empty_like(tq)
    torch.cuda.synchronize()
    gc.collect()
    times = []
    t_warm = time.perf_counter()
    rep = 0
    while True:                               # untimed passes until the chip has worked for 60 ms, then the timed one; the pages
        last = rep >= 1 and (time.perf_counter() - t_warm) >= 0.06      # are simply overwritten again
        rep += 1
        times.clear()
        with no_gc():
            for t in range(n_steps):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                sgc.sgc_decode_step_batched(s.ctx, s.cache, s.plan, layer, t, tq.data_ptr(), tk.data_ptr(), tv.data_ptr(),
                                            to.data_ptr(), None, stream)
                e1.record()
                times.append((e0, e1))
            torch.cuda.synchronize()
        if last:
            break
    ms = [a.elapsed_time(b) for a, b in times]
    live = w.suffix_len > 0
    S = w.suffix_len[live].astype(np.float64)
    P = w.prefix_len[w.labels[live]].astype(np.float64)
    t_mid = (n_steps - 1) / 2.0
    kvb = 2.0 * w.n_kv_heads * w.head_dim                         # K and V elements per token
    used = np.unique(w.labels[live])
    cache_bytes = float(w.prefix_len[used].sum()) * kvb * w.kv_bytes()
    own_bytes = float(np.sum(S + t_mid + 1)) * kvb * 2
    io_bytes = float(live.sum()) * (2 * w.n_q_heads + 2 * w.n_kv_heads) * w.head_dim * 2
    alg_bytes = cache_bytes + own_bytes + io_bytes
    flop = float(4.0 * w.n_q_heads * w.head_dim * np.sum(P + S + t_mid + 1))
    mean_ms = float(np.mean(ms))
    per_query_read = float(np.sum(P)) * kvb * w.kv_bytes() + own_bytes + io_bytes     # without the sharing
    return {"steps": n_steps, "ms_per_step": mean_ms, "ms_per_step_min": float(np.min(ms)),
            "us_per_query_step": mean_ms * 1e3 / max(int(live.sum()), 1),
            "algorithmic_bytes_per_step": alg_bytes, "flop_per_step": flop,
            "roofline": {"bound": "hbm", "achieved": alg_bytes / (mean_ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                         "frac": alg_bytes / (mean_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                         "traffic": PROFILED_DECODE_STEP_BYTES.get(w.name, (None, None))[0],
                         "traffic_source": PROFILED_DECODE_STEP_BYTES.get(w.name, (None, None))[1]},
            "bytes_if_every_query_read_its_prefix": per_query_read}


def layer_measurement(s, w, layer, d_model, reps, stream):
    """The attention layer around the kernel (QKV projection with the fused page-writing epilogue, attention from
    the projected keys, output projection) on the same workload: per-call times from HIP events on the launch
    stream.  Random weights and hidden states stand in for a trained model's."""
    import torch
    from paper_2505_10951_amd import sgc
    from paper_2505_10951_amd.harness import to_device
    all_clusters = list(range(w.n_clusters))
    if sgc.sgc_cache_free_pages(s.cache) == sgc.sgc_cache_total_pages(s.cache):
        for c in all_clusters:
            sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(w.prefix_len[c]))
    w_qkv, w_o = w.layer_weights(d_model, layer)
    dwq, dwo = to_device(w_qkv, w.io_dtype), to_device(w_o, w.io_dtype)
    dpx = [to_device(w.prefix_x(c, d_model, layer), w.io_dtype) for c in all_clusters]
    dx = to_device(w.suffix_x(d_model, layer), w.io_dtype)
    T, nq = dx.shape[0], w.n_q_heads * w.head_dim
    n_qkv = nq + 2 * w.n_kv_heads * w.head_dim
    dq = torch.empty((T, nq), dtype=dx.dtype, device=dx.device)
    do = torch.empty_like(dq)
    dy = torch.empty((T, d_model), dtype=dx.dtype, device=dx.device)
    px_ptrs = [t.data_ptr() for t in dpx]

    def timed(fn):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        return e0, e1

    calls = {
        "qkv_prefix": lambda: sgc.sgc_project_qkv_prefix_batched(s.ctx, s.cache, all_clusters, layer, px_ptrs, dwq.data_ptr(),
                                                                 d_model, None, stream),
        "qkv_suffix": lambda: sgc.sgc_project_qkv_suffix(s.ctx, s.cache, s.plan, layer, dx.data_ptr(), dwq.data_ptr(), d_model,
                                                         dq.data_ptr(), stream),
        "attention": lambda: sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, layer, dq.data_ptr(), None, None,
                                                            do.data_ptr(), None, stream),
        "out": lambda: sgc.sgc_project_out(s.ctx, do.data_ptr(), dwo.data_ptr(), d_model, T, dy.data_ptr(), stream),
    }
    calls["qkv_prefix"]()
    s.assign(w.labels, w.suffix_len)
    s.upload_plan()
    evs = {k: [] for k in calls}
    gc.collect()
    t_warm = time.perf_counter()
    n_warm = 0
    while n_warm < 2 or (time.perf_counter() - t_warm) < 0.06:      # untimed rounds until the chip's clocks are up
        for fn in calls.values():
            fn()
        torch.cuda.synchronize()
        n_warm += 1
    with no_gc():
        for rep in range(reps):
            for name, fn in calls.items():
                evs[name].append(timed(fn))
        torch.cuda.synchronize()
    ms = {k: float(np.mean([a.elapsed_time(b) for a, b in v])) for k, v in evs.items()}
    P_total = float(w.prefix_len.sum())
    flop = {"qkv_prefix": 2.0 * P_total * d_model * (n_qkv - nq),          # the prompt's queries are not needed here
            "qkv_suffix": 2.0 * T * d_model * n_qkv, "attention": w.flops(), "out": 2.0 * T * nq * d_model}
    peak = PEAK_TFLOPS[w.io_dtype]
    per = {k: {"ms": ms[k], "tflops": flop[k] / (ms[k] * 1e-3) / 1e12} for k in calls}
    suffix_ms = ms["qkv_suffix"] + ms["attention"] + ms["out"]
    suffix_flop = flop["qkv_suffix"] + flop["attention"] + flop["out"]
    gemm = per["qkv_suffix"]
    return {"d_model": d_model, "calls": per,
            "suffix_layer_ms": suffix_ms, "suffix_layer_tflops": suffix_flop / (suffix_ms * 1e-3) / 1e12,
            "suffix_layer_us_per_query": suffix_ms * 1e3 / max(w.n_queries, 1),
            "roofline": {"kernel": "proj_gemm_kernel<true> (QKV projection, keys and values written into suffix pages)",
                         "bound": "mfma" if w.io_dtype == "bf16" else "alu", "achieved": gemm["tflops"], "peak": peak,
                         "unit": "TFLOP/s", "frac": gemm["tflops"] / peak,
                         "traffic": PROFILED_QKV_GEMM_BYTES.get((w.name, d_model), (None, None))[0],
                         "traffic_source": PROFILED_QKV_GEMM_BYTES.get((w.name, d_model), (None, None))[1]}}


def host_steps(s, w, ms_per_step: float):
    """The host-side steps in front of the prefill (SubGCache Sec. 3.2 and 3.3; the paper puts "cluster processing" below
    2.1 % / 6 % of a query's latency): agglomerative clustering of the batch's query embeddings under Table 3's linkages,
    the per-cluster union of the retrieved subgraphs, and the query -> cluster -> cache mapping, each as the median of five
    calls on the same workload (synthetic embeddings and subgraphs with the workload's cluster structure)."""
    from paper_2505_10951_amd import sgc
    emb = w.query_embeddings(dim=64)
    node_lists, edge_lists = w.retrieved_subgraphs()
    fresh = sgc.sgc_cache_free_pages(s.cache) == sgc.sgc_cache_total_pages(s.cache)
    if fresh:                                   # the mapping needs the clusters' caches to exist (host-side allocation only)
        for c in range(w.n_clusters):
            sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(w.prefix_len[c]))

    def med_us(fn):
        ts = []
        for _ in range(5):
            t0 = time.perf_counter()
            fn()
            ts.append(time.perf_counter() - t0)
        return float(np.median(ts) * 1e6)

    out = {"n_queries": int(w.n_queries), "embedding_dim": 64,
           "cluster_queries_us": {name: med_us(lambda name=name: sgc.sgc_cluster_queries(s.ctx, emb, w.n_clusters, name))
                                  for name in sgc.LINKAGES},
           "union_subgraphs_us": med_us(lambda: sgc.sgc_union_subgraphs(s.ctx, w.labels, w.n_clusters, node_lists, edge_lists)),
           "assign_clusters_us": med_us(lambda: s.assign(w.labels, w.suffix_len))}
    out["labels_recovered"] = bool(_same_partition(sgc.sgc_cluster_queries(s.ctx, emb, w.n_clusters, "ward"), w.labels))
    total = out["cluster_queries_us"]["ward"] + out["union_subgraphs_us"] + out["assign_clusters_us"]
    out["share_of_a_step"] = total / (ms_per_step * 1e3)
    out["us_per_query"] = total / max(int(w.n_queries), 1)
    if fresh:
        for c in range(w.n_clusters):
            sgc.sgc_cache_free_cluster(s.ctx, s.cache, c)
    return out


def _same_partition(a, b) -> bool:
    """Two labelings describe the same partition (cluster numbers may differ)."""
    a, b = np.asarray(a), np.asarray(b)
    pairs = set(zip(a.tolist(), b.tolist()))
    return len(pairs) == len(set(a.tolist())) == len(set(b.tolist()))


def other_config(index: int, steps: int, warmup: int, threads: int, kernel=None):
    """One of the other benchmark configurations: its batched suffix prefill launched `steps` times (caches filled
    and the plan uploaded beforehand; kernel durations from the library's HIP events on the launch stream), the
    kernel's roofline figures, and the error against the oracle on two of its queries."""
    import torch
    from paper_2505_10951_amd import sgc, workloads
    from paper_2505_10951_amd.harness import Session, to_device
    w = workloads.config(index)
    layer = 0
    q, k, v = w.suffix_qkv(layer, threads=threads)
    clusters = list(range(w.n_clusters))
    if kernel is None:        # an fp8 cache over long prompts: first product on the e4m3 codes
        kernel = sgc.SGC_KERNEL_MFMA_FP8 if w.kv_dtype == "fp8_e4m3" else sgc.SGC_KERNEL_AUTO
    with Session(w, kernel=kernel) as s:
        stream = s.stream
        for c in clusters:
            sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(w.prefix_len[c]))
            pk, pv = w.prefix_kv(c, layer)
            dpk, dpv = to_device(pk, w.io_dtype), to_device(pv, w.io_dtype)
            sgc.sgc_prefix_prefill(s.ctx, s.cache, c, layer, None, dpk.data_ptr(), dpv.data_ptr(), None, None,
                                   int(w.prefix_len[c]), stream)
            torch.cuda.synchronize()
            del dpk, dpv
        dq, dk, dv = (to_device(x, w.io_dtype) for x in (q, k, v))
        do = torch.empty_like(dq)
        s.assign(w.labels, w.suffix_len)
        s.upload_plan()
        def launch():
            sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, layer, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
                                           do.data_ptr(), None, stream)
        # untimed launches until the chip has worked for 60 ms (its clocks are up by then), at least `warmup` of them
        gc.collect()
        t0 = time.perf_counter()
        n_warm = 0
        while n_warm < warmup or (time.perf_counter() - t0) < 0.06:
            launch()
            torch.cuda.synchronize()
            n_warm += 1
        per_launch = (time.perf_counter() - t0) / n_warm
        steps = int(min(100, max(steps, np.ceil(0.06 / per_launch))))
        warmup = n_warm
        sgc.sgc_timing_enable(s.ctx, True)
        with no_gc():
            for i in range(steps):
                launch()
            torch.cuda.synchronize()
        kernel_ms = [sgc.sgc_timing_get(s.ctx, back) for back in range(steps)]
        info = sgc.sgc_plan_get_info(s.ctx, s.plan)
        # two queries against the oracle: the first of the largest and of the smallest cluster
        sizes = np.bincount(w.labels, minlength=w.n_clusters)
        picks = sorted({int(np.flatnonzero(w.labels == int(np.argmax(sizes)))[0]),
                        int(np.flatnonzero(w.labels == int(np.argmin(np.where(sizes > 0, sizes, sizes.max() + 1))))[0])})
        _, _, o_ref, rows = oracle_on_queries(w, picks, layer)
        o_rows = do[torch.from_numpy(rows).to(do.device)].to(torch.float32).cpu().numpy()
        for c in clusters:
            sgc.sgc_cache_free_cluster(s.ctx, s.cache, c)
    attn_ms = float(np.mean([b for _, b in kernel_ms]))
    ingest_ms = float(np.mean([a for a, _ in kernel_ms]))
    mfma = w.io_dtype == "bf16" and w.head_dim == 128
    peak = PEAK_TFLOPS["bf16" if mfma else "f32"]
    path = "16-bit matrix-core products (binary16 QK^T, bf16 PV)" if mfma else "fp32 matrix-core products"
    achieved = w.flops() / (attn_ms * 1e-3) / 1e12
    extra = {}
    if kernel == sgc.SGC_KERNEL_MFMA_FP8:
        # half the flops (QK^T) run at the fp8 matrix-core rate, half (PV) at the bf16 rate
        peak = 2.0 / (1.0 / PEAK_TFLOPS["fp8"] + 1.0 / PEAK_TFLOPS["bf16"])
        path = "QK^T on the cache's e4m3 codes (fp8 matrix-core rate, query rows quantised to e4m3), PV on bf16"
        extra = {"frac_of_bf16_peak": achieved / PEAK_TFLOPS["bf16"], "frac_of_fp8_peak": achieved / PEAK_TFLOPS["fp8"],
                 "peak_is": "harmonic mean of the fp8 and bf16 dense peaks (half the flops at each rate)"}
    elif w.kv_dtype == "fp8_e4m3":
        path = "e4m3 codes widened to 16-bit on their way into LDS, 16-bit matrix-core products"
    prof = PROFILED_HBM_BYTES_PER_LAUNCH.get((w.name, "fp8_first_product" if kernel == sgc.SGC_KERNEL_MFMA_FP8 else "16bit"))
    return {"workload": f"configs[{index}] {w.name}: Hq {w.n_q_heads} Hkv {w.n_kv_heads} d {w.head_dim}, {w.n_clusters} clusters, "
                        f"prefix {int(w.prefix_len.min())}-{int(w.prefix_len.max())}, {w.n_queries} queries, "
                        f"{w.total_suffix_tokens} suffix tokens, io {w.io_dtype}, kv {w.kv_dtype}",
            "timed": f"{steps} suffix launches after {warmup} untimed, caches and plan resident",
            "n_tiles": info.n_tiles, "suffix_flop": w.flops(),
            "attention_kernel_ms": attn_ms, "attention_kernel_ms_min": float(np.min([b for _, b in kernel_ms])),
            "attention_kernel_ms_median": float(np.median([b for _, b in kernel_ms])),
            "before_attention_kernel_ms": ingest_ms, "suffix_call_ms": attn_ms + ingest_ms,
            "us_per_query": (attn_ms + ingest_ms) * 1e3 / w.n_queries,
            "roofline": {"kernel": "attn_mfma_kernel (batched suffix prefill)" if mfma else "attn_generic_kernel (fp32 matrix cores)",
                         "path": path, "bound": "mfma" if mfma else "alu", "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                         "frac": achieved / peak, "frac_of_call": w.flops() / ((attn_ms + ingest_ms) * 1e-3) / 1e12 / peak,
                         "traffic": prof[0] if prof else None, "traffic_source": prof[1] if prof else None,
                         "algorithmic_bytes": w.algorithmic_bytes(),
                         "hbm_gbs_algorithmic": w.algorithmic_bytes() / (attn_ms * 1e-3) / 1e9,
                         "co_limits": co_limits(achieved) if mfma else None, **extra},
            **({"cpu_baseline_one_thread": oracle_one_thread(index)} if index == 0 else {}),
            "error": error_against_oracle(o_rows, o_ref, w.kv_dtype, f"queries {picks}: all heads, all rows")}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=50)
    ap.add_argument("--config", type=int, default=1, help="which of the five benchmark configurations, 0-4 (default 1: Llama-3-8B-shaped layer)")
    ap.add_argument("--cpu-budget", type=float, default=15.0, help="seconds of oracle time for the CPU baseline (0 = skip)")
    ap.add_argument("--wait-every-step", action="store_true",
                    help="wait for the GPU after every timed step (a step's latency) instead of enqueueing the steps back to back "
                         "between the two synchronisations that bracket the timed region")
    ap.add_argument("--pipelined", action="store_true", help=argparse.SUPPRESS)      # the default; accepted for older command lines
    ap.add_argument("--no-host-steps", dest="host_steps", action="store_false",
                    help="skip the timing of the host steps in front of the prefill (clustering, subgraph union, assignment)")
    ap.add_argument("--kernel-timing-period", type=int, default=4,
                    help="HIP events around the suffix kernels of every n-th timed step (1 = every step)")
    ap.add_argument("--suffix-only", action="store_true", help="time only the batched suffix launch (profiling aid)")
    ap.add_argument("--decode-steps", type=int, default=32,
                    help="after the timed steps, time this many batched decode steps on the same workload (0 = skip)")
    ap.add_argument("--layer-d-model", type=int, default=-1,
                    help="model width of the attention-layer measurement (-1: n_q_heads * head_dim, 0: skip)")
    ap.add_argument("--layer-reps", type=int, default=10)
    ap.add_argument("--other-configs", type=str, default="auto",
                    help="comma-separated indices of further configurations whose suffix launch is timed and reported "
                         "under \"configs\" (auto: 0,2,3,4 when the headline is configs[1], else none; none: skip)")
    ap.add_argument("--kernel", choices=["auto", "mfma", "mfma_fp8", "generic"], default="auto",
                    help="attention kernel of the headline configuration (auto: the matrix-core kernel where it covers the shape, "
                         "with the first product on the e4m3 codes when the cache is fp8)")
    ap.add_argument("--queries-per-cluster", type=int, default=None,
                    help="another batch size for the headline configuration, everything else as it is (sweeps of the launch size; "
                         "the suffix-length range is the configuration's observed one, so the default size need not reproduce it exactly)")
    ap.add_argument("--other-steps", type=int, default=5,
                    help="timed suffix launches per further configuration, at least (as many as fill 60 ms, at most 100)")
    ap.add_argument("--settle-ms", type=float, default=100.0,
                    help="before the warm-up steps, run untimed steps for this long: the chip raises its clocks over the first tens of "
                         "milliseconds of work, and a handful of half-millisecond steps would be timed on the way up (0 = skip)")
    ap.add_argument("--repeat-launches", type=int, default=100,
                    help="after the timed steps, launch the suffix call this many times back to back (after 60 ms of untimed ones) and report "
                         "median and minimum kernel time (0 = skip, at most 128)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run ten 256 MiB device copies and exit (counter calibration under rocprofv3 --pmc)")
    args = ap.parse_args()
    args.pipelined = not args.wait_every_step
    if args.gpus != 1:
        print(f"bench.py: this build runs on ONE GPU (no collectives, no sharding); --gpus {args.gpus} is not supported",
              file=sys.stderr)
        return 2

    import torch
    from paper_2505_10951_amd import sgc, workloads
    from paper_2505_10951_amd.harness import Session, to_device

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 2
    if args.copy_calibration:
        return copy_calibration()
    w = workloads.config(args.config, queries_per_cluster=args.queries_per_cluster)
    layer = 0
    t_gen = time.perf_counter()
    gen_threads = min(16, os.cpu_count() or 1)
    q, k, v = w.suffix_qkv(layer, threads=gen_threads)
    pkv = [w.prefix_kv(c, layer) for c in range(w.n_clusters)]
    pq = [w.prefix_q(c, layer) for c in range(w.n_clusters)]
    t_gen = time.perf_counter() - t_gen

    kinds = {"auto": sgc.SGC_KERNEL_MFMA_FP8 if w.kv_dtype == "fp8_e4m3" else sgc.SGC_KERNEL_AUTO, "mfma": sgc.SGC_KERNEL_MFMA,
             "mfma_fp8": sgc.SGC_KERNEL_MFMA_FP8, "generic": sgc.SGC_KERNEL_GENERIC}
    s = Session(w, kernel=kinds[args.kernel])
    dq, dk, dv = (to_device(x, w.io_dtype) for x in (q, k, v))
    do = torch.empty_like(dq)
    dpk = [to_device(a, w.io_dtype) for a, _ in pkv]
    dpv = [to_device(b, w.io_dtype) for _, b in pkv]
    dpq = [to_device(a, w.io_dtype) for a in pq]
    dpo = [torch.empty_like(a) for a in dpq]
    torch.cuda.synchronize()
    stream = s.stream
    labels, slen = w.labels, w.suffix_len
    all_clusters = list(range(w.n_clusters))
    pq_ptrs, pk_ptrs, pv_ptrs, po_ptrs = ([t.data_ptr() for t in ts] for ts in (dpq, dpk, dpv, dpo))
    sgc.sgc_timing_enable(s.ctx, True)

    def step(wait: bool):
        if not args.suffix_only or s.plan is None:
            for c in range(w.n_clusters):
                sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(w.prefix_len[c]))
            sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, all_clusters, layer, pq_ptrs, pk_ptrs, pv_ptrs, po_ptrs, None, stream)
            s.assign(labels, slen)
            s.upload_plan()
        sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, layer, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
                                       do.data_ptr(), None, stream)
        if not args.suffix_only:
            # Everything runs on one stream: the next step's ingest, which reuses these pages, is ordered behind
            # this step's attention kernels, so the pages are handed back while the GPU still works.
            for c in range(w.n_clusters):
                sgc.sgc_cache_free_cluster(s.ctx, s.cache, c)
        if wait:
            torch.cuda.synchronize()

    # Default: the K timed steps are enqueued back to back on the one stream, between the two synchronisations that bracket
    # the timed region (throughput).  --wait-every-step waits for the GPU after every step (a step's latency): 5-6 % slower,
    # the kernels' own times the same.  The other mode is run too, after the timed steps, and reported as "other_mode".
    def timed_loop(wait: bool):
        torch.cuda.synchronize()
        with no_gc():
            t_start = time.perf_counter()
            for _ in range(args.steps):
                step(wait)
            torch.cuda.synchronize()
            return (time.perf_counter() - t_start) / args.steps * 1e3

    gc.collect()
    t_settle = time.perf_counter()
    n_settle = 0
    while (time.perf_counter() - t_settle) * 1e3 < args.settle_ms:
        step(True)
        n_settle += 1
    for _ in range(args.warmup):
        step(not args.pipelined)
    torch.cuda.synchronize()
    # The library's HIP events around the suffix launch's kernels cost the stream about 8 us per launch (2 % of a step), so
    # inside the timed steps every `period`-th launch carries them: the kernel's duration is a sample of the timed region,
    # the step time is taken with three quarters of the steps unobserved.
    period = max(1, args.kernel_timing_period)
    n_sampled = min((args.steps + period - 1) // period, 128)          # (the library keeps the last 128)
    sgc.sgc_timing_enable(s.ctx, period)        # also restarts the library's count of timed launches
    ms_per_step = timed_loop(not args.pipelined)
    kernel_ms = [sgc.sgc_timing_get(s.ctx, back) for back in range(n_sampled)]
    kern_ms = float(np.mean([a + b for a, b in kernel_ms]))                    # ingest + attention
    kern_ms_min = float(np.min([a + b for a, b in kernel_ms]))
    ingest_ms = float(np.mean([a for a, _ in kernel_ms]))
    attn_ms = float(np.mean([b for _, b in kernel_ms]))                        # the dominant kernel alone
    attn_ms_min = float(np.min([b for _, b in kernel_ms]))
    attn_ms_median = float(np.median([b for _, b in kernel_ms]))
    other = None
    if not args.suffix_only:
        sgc.sgc_timing_enable(s.ctx, period)
        other_ms = timed_loop(bool(args.pipelined))
        other_kernel = [sgc.sgc_timing_get(s.ctx, back)[1] for back in range(n_sampled)]
        other = {"mode": "host waits after every step" if args.pipelined else "steps enqueued back to back",
                 "ms_per_step": other_ms, "attention_kernel_ms": float(np.mean(other_kernel))}

    o_host = do.to(torch.float32).cpu().numpy()          # what the last timed step wrote, for the error figures
    repeat = None
    if not args.suffix_only and args.repeat_launches > 0:
        # the suffix call alone, launched back to back with caches and plan resident: 60 ms of untimed launches, then the timed ones
        for c in range(w.n_clusters):
            sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(w.prefix_len[c]))
        sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, all_clusters, layer, pq_ptrs, pk_ptrs, pv_ptrs, po_ptrs, None, stream)
        s.assign(labels, slen)
        s.upload_plan()
        n_rep = min(args.repeat_launches, 128)
        def launch():
            sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, layer, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
                                           do.data_ptr(), None, stream)
        gc.collect()
        t_warm, n_untimed = time.perf_counter(), 0
        while n_untimed < 20 or (time.perf_counter() - t_warm) < 0.06:      # the chip has been idle: 60 ms of launches first
            for _ in range(20):
                launch()
            torch.cuda.synchronize()
            n_untimed += 20
        sgc.sgc_timing_enable(s.ctx, True)
        with no_gc():
            for _ in range(n_rep):
                launch()
            torch.cuda.synchronize()
        rep_ms = [sgc.sgc_timing_get(s.ctx, back)[1] for back in range(n_rep)]
        for c in range(w.n_clusters):
            sgc.sgc_cache_free_cluster(s.ctx, s.cache, c)
        med = float(np.median(rep_ms))
        repeat = {"launches": n_rep, "untimed_before": n_untimed, "mode": "the suffix call repeated back to back, caches and plan resident",
                  "attention_kernel_ms_median": med, "attention_kernel_ms_min": float(np.min(rep_ms)),
                  "attention_kernel_ms_mean": float(np.mean(rep_ms)),
                  "roofline_frac_median": w.flops() / (med * 1e-3) / 1e12 / PEAK_TFLOPS[w.io_dtype]}
    fl_suffix = w.flops()
    fl_step = fl_suffix + (0.0 if args.suffix_only else prefix_flops(w))
    info = sgc.sgc_plan_get_info(s.ctx, s.plan)
    dtype = w.io_dtype
    peak = PEAK_TFLOPS[dtype]
    achieved = fl_suffix / (attn_ms * 1e-3) / 1e12
    prof = PROFILED_HBM_BYTES_PER_LAUNCH.get((w.name, "fp8_first_product" if kinds[args.kernel] == sgc.SGC_KERNEL_MFMA_FP8 else "16bit"))
    mfma = dtype == "bf16" and w.head_dim == 128
    out = {
        "metric": "suffix-prefill attention TFLOP/s (% MFMA peak) and us/query vs CPU oracle",
        "value": fl_step / (ms_per_step * 1e-3) / 1e12,
        "unit": "TFLOP/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": dtype, "data": "synthetic",
        "config": {"workload": f"configs[{args.config}] {w.name}: Hq {w.n_q_heads} Hkv {w.n_kv_heads} d {w.head_dim}, "
                               f"{w.n_clusters} clusters, prefix {int(w.prefix_len.min())}-{int(w.prefix_len.max())}, "
                               f"{w.n_queries} queries, {w.total_suffix_tokens} suffix tokens, kv {w.kv_dtype}",
                   "step": "suffix launch only" if args.suffix_only else
                           "alloc + batched prefix prefill (ingest + causal attention) + assign/plan upload + batched suffix prefill + free",
                   "tile_rows": info.tile_rows, "n_tiles": info.n_tiles,
                   "settle": f"{n_settle} untimed steps ({args.settle_ms:g} ms) before the warm-up steps",
                   "kernel_timing": f"HIP events around the suffix kernels of every {period}. timed step ({n_sampled} launches)"},
        "step_flop": fl_step, "suffix_flop": fl_suffix,
        "suffix_launch_ms": kern_ms, "suffix_launch_ms_min": kern_ms_min,
        # (what the call launches before the attention kernel; where that is nothing, the distance of two event records, 5 us)
        "before_attention_kernel_ms": ingest_ms, "attention_kernel_ms": attn_ms, "attention_kernel_ms_min": attn_ms_min,
        "attention_kernel_ms_median": attn_ms_median,
        "us_per_query": ms_per_step * 1e3 / w.n_queries,
        "suffix_us_per_query": kern_ms * 1e3 / w.n_queries,
        "pct_mfma_peak_step": 100.0 * fl_step / (ms_per_step * 1e-3) / 1e12 / peak,
        "roofline": {"kernel": "attn_mfma_kernel (batched suffix prefill)" if mfma else "attn_generic_kernel (fp32 matrix cores)",
                     "bound": "mfma" if mfma else "alu", "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                     "frac": achieved / peak,
                     # the whole call (what is launched before the attention kernel + the attention kernel) against the same peak
                     "frac_of_call": fl_suffix / (kern_ms * 1e-3) / 1e12 / peak,
                     "traffic": prof[0] if prof else None, "traffic_source": prof[1] if prof else None,
                     "algorithmic_bytes": w.algorithmic_bytes(),
                     "hbm_gbs_algorithmic": w.algorithmic_bytes() / (attn_ms * 1e-3) / 1e9,
                     "hbm_frac_algorithmic": w.algorithmic_bytes() / (attn_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                     "co_limits": co_limits(achieved) if mfma else None},
        "paper_context": "TTFT reduction up to 6.68x, PFTT up to 15.49x (Table 2; 2x A100-SXM4-40GB, precision not stated); end-to-end LLM latencies, not this kernel",
        "input_gen_s": t_gen,
    }
    out["config"]["mode"] = "steps enqueued back to back" if args.pipelined else "host waits after every step"
    if other is not None:
        other["value"] = fl_step / (other["ms_per_step"] * 1e-3) / 1e12
        other["roofline_frac"] = fl_suffix / (other["attention_kernel_ms"] * 1e-3) / 1e12 / peak
        out["other_mode"] = other
    if repeat is not None:
        out["repeat_launches"] = repeat
    d_model = w.n_q_heads * w.head_dim if args.layer_d_model < 0 else args.layer_d_model
    if d_model > 0 and not args.suffix_only:
        out["layer"] = layer_measurement(s, w, layer, d_model, args.layer_reps, stream)
        torch.cuda.synchronize()
        for c in range(w.n_clusters):
            sgc.sgc_cache_free_cluster(s.ctx, s.cache, c)
    if args.decode_steps > 0 and dtype == "bf16":
        out["decode"] = decode_measurement(s, w, layer, args.decode_steps, dq, dk, dv, do, all_clusters,
                                           pq_ptrs, pk_ptrs, pv_ptrs, po_ptrs, stream)
    if not args.suffix_only and args.host_steps:
        out["host_steps"] = host_steps(s, w, ms_per_step)
    s.close()
    if args.cpu_budget > 0:
        out["cpu_baseline"], rows, o_ref = cpu_baseline(w, args.cpu_budget)
        out["gpu_over_cpu"] = achieved / out["cpu_baseline"]["value"]
        # the oracle's outputs for its sample against what the last timed step left in o (outside the timed region)
        err = error_against_oracle(o_host[rows], o_ref, w.kv_dtype, out["cpu_baseline"]["sample"])
        out["max_abs_err"], out["rel_err"], out["error"] = err["max_abs_err"], err["rel_err"], err
    others = args.other_configs
    if others == "auto":
        others = "0,2,3,4" if (args.config == 1 and not args.suffix_only) else "none"
    if others != "none":
        del o_host, dq, dk, dv, do, dpk, dpv, dpq, dpo
        torch.cuda.empty_cache()
        out["configs"] = [other_config(int(i), args.other_steps, 2, gen_threads) for i in others.split(",") if i.strip()]
        if "4" in [i.strip() for i in others.split(",")]:
            # the same configuration with the first product on 16-bit operands: what the fp8 first product buys
            alt = other_config(4, args.other_steps, 2, gen_threads, kernel=sgc.SGC_KERNEL_MFMA)
            alt["workload"] += " [comparison: 16-bit first product]"
            out["configs"].append(alt)
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
