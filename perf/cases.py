"""The work that programs have libsgc do, as cases that can be timed and compared: cluster-shared prefill of a batch,
suffix prefill over resident caches, batched decode, and the attention layer with its projections.

A case is a dict of plain values.  `kind` says which calls a pass makes:
  serve   a batch from nothing: pages for every cluster, the prompts' prefill (keys stored, causal attention), the
          query -> cluster -> cache mapping, the suffix prefill of every query, pages handed back
  suffix  the suffix prefill alone, layer by layer, with the caches filled and the plan made beforehand
  decode  `steps` generated tokens per query behind a suffix prefill that has run
  layer   hidden states in, hidden states out: projections, attention and output projection of prompts and batch
The lengths and labels of a batch follow from the case (`shape`), its values from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_10951_amd import sgc, workloads

DEVICE = "cuda:0"
KERNELS = {"auto": sgc.SGC_KERNEL_AUTO, "mfma_fp8": sgc.SGC_KERNEL_MFMA_FP8}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(kind, hq, hkv, d, clusters, prefix, queries, suffix, **more):
    c = {"kind": kind, "hq": hq, "hkv": hkv, "d": d, "clusters": clusters, "prefix_lo": prefix[0], "prefix_hi": prefix[1],
         "queries": queries, "suffix_lo": suffix[0], "suffix_hi": suffix[1], "zipf": False, "io": "bf16", "kv": "bf16",
         "kernel": "auto", "rope": 500000.0, "outlier": 1.0, "layers": 1, "steps": 0, "d_model": 0, "lse": False, "shape": 1}
    c.update(more)
    return c


def listed():
    return [
        # one question over one retrieved subgraph: the smallest call, launches and host work
        _case("serve", 32, 8, 128, 1, (411, 411), 1, (23, 23), name="one_question"),
        # the paper's own batch size: 100 one-sentence questions, ten prompts of up to about a thousand tokens, a few layers
        _case("serve", 32, 8, 128, 10, (150, 1000), 100, (8, 40), layers=4, name="paper_batch"),
        # the benchmark's batch: a Llama-3-8B-shaped layer, keys with outlier channels
        _case("serve", 32, 8, 128, 10, (1024, 1024), 320, (16, 64), outlier=8.0, name="llama3_batch"),
        # the fp32 layer with small heads
        _case("serve", 4, 4, 64, 2, (192, 256), 16, (16, 32), io="f32", kv="f32", rope=10000.0, name="tiny_f32"),
        # an fp8 cache filled from prompts of several thousand tokens and used for a batch
        _case("serve", 64, 8, 128, 6, (2000, 8000), 96, (32, 256), kv="fp8_e4m3", name="fp8_prompts"),
        # Llama-2-7B-shaped: no head groups, ragged prompts, Zipf-sized clusters; the log-sum-exp goes out too
        _case("suffix", 32, 32, 128, 16, (1024, 4096), 1024, (24, 96), zipf=True, rope=10000.0, lse=True, name="ragged_mha"),
        # several layers of the 32-layer stack over a resident cache (the layers are alike)
        _case("suffix", 32, 8, 128, 16, (4096, 4096), 256, (128, 128), layers=4, name="stack"),
        # 70B-shaped layer over long fp8 prompts, first product on the codes: the largest
        _case("suffix", 64, 8, 128, 8, (16384, 16384), 1024, (32, 256), kv="fp8_e4m3", kernel="mfma_fp8", name="long_fp8"),
        # generation: 32 tokens for every query of the benchmark's batch
        _case("decode", 32, 8, 128, 10, (1024, 1024), 320, (16, 64), outlier=8.0, steps=32, name="decode"),
        # generation for a handful of queries over one longer prompt
        _case("decode", 32, 8, 128, 1, (3001, 3001), 5, (11, 47), steps=16, name="decode_few"),
        # the attention layer around the benchmark's batch
        _case("layer", 32, 8, 128, 10, (1024, 1024), 320, (16, 64), d_model=4096, name="layer"),
        # the same layer for one short prompt and a few questions
        _case("layer", 32, 8, 128, 1, (300, 300), 6, (12, 40), d_model=4096, name="layer_few"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# what a drawn case may cost at most, per kind (flop of a pass)
_CAP = {"serve": 4e12, "suffix": 2e13, "decode": 2e11, "layer": 6e12}


def draw(rng):
    kind = rng.choice(["serve", "serve", "suffix", "suffix", "decode", "layer"])
    small_heads = kind == "serve" and rng.random() < 0.25
    if small_heads:             # what the matrix-core kernel does not cover: fp32, heads of 64 channels
        io, d = rng.choice([("f32", 64), ("f32", 128), ("bf16", 64)])
        hq, hkv = rng.choice([(4, 4), (8, 2), (16, 4)])
        kv, kernel = io, "auto"
        clusters, queries = _log(rng, 1, 6), _log(rng, 1, 40)
        prefix, suffix = _log(rng, 60, 600), _log(rng, 4, 40)
    else:
        io, d = "bf16", 128
        hq, hkv = rng.choice([(32, 8), (32, 8), (32, 32), (64, 8), (8, 2)])
        kv, kernel = rng.choice([("bf16", "auto")] * 3 + [("fp8_e4m3", "auto"), ("fp8_e4m3", "mfma_fp8")])
        if kind == "layer":
            kv, kernel = rng.choice([("bf16", "auto")] * 4 + [("fp8_e4m3", "auto")])
        clusters = _log(rng, 1, 24)
        queries = clusters * _log(rng, 1, 64)
        prefix = _log(rng, 120, 12000 if kind in ("suffix", "decode") else 4000)
        suffix = _log(rng, 8, 200)
    c = _case(kind, hq, hkv, d, clusters, (max(1, prefix * rng.randint(40, 100) // 100), prefix), queries,
              (max(1, suffix * rng.randint(20, 100) // 100), suffix), io=io, kv=kv, kernel=kernel, zipf=rng.random() < 0.3,
              rope=rng.choice([10000.0, 500000.0]), outlier=rng.choice([1.0, 1.0, 8.0]) if kind != "layer" else 1.0,
              lse=kind != "layer" and rng.random() < 0.25, shape=rng.randint(1, 1 << 20))
    if kind in ("serve", "suffix") and not small_heads:
        c["layers"] = rng.choice([1, 1, 2, 4])
    if kind == "decode":
        c["steps"] = rng.choice([4, 8, 16, 32])
    if kind == "layer":
        c["d_model"] = rng.choice([1024, 2048, 4096, 4096, 5120])
    if kernel == "mfma_fp8":    # meant for long prompts and plain keys: its e4m3 query rows need many keys to average over
        c["outlier"] = 1.0
        c["prefix_lo"] = max(4000, c["prefix_lo"])
        c["prefix_hi"] = max(c["prefix_lo"], c["prefix_hi"])
    cap = 1e10 if small_heads else _CAP[kind]
    while c["queries"] > 1 and (work(c)["flops"] > cap or c["queries"] * c["suffix_hi"] * hq > 12_000_000):
        c["queries"] = max(1, c["queries"] * 2 // 3)
        c["clusters"] = max(1, min(c["clusters"], c["queries"]) * 4 // 5)
    return c


def _structure(case):
    """The batch's lengths and labels (no values): a Workload that only its integers are taken from."""
    rng = np.random.default_rng(case["shape"])
    nc, nq = case["clusters"], case["queries"]
    prefix_len = rng.integers(case["prefix_lo"], case["prefix_hi"] + 1, size=nc).astype(np.int32)
    if case["zipf"]:
        sizes = workloads.zipf_cluster_sizes(nc, nq)
        rng.shuffle(sizes)
    else:
        sizes = np.full(nc, nq // nc, dtype=np.int32)
        sizes[: nq - int(sizes.sum())] += 1
    return workloads.custom(case["kind"], n_q_heads=case["hq"], n_kv_heads=case["hkv"], head_dim=case["d"], rope_base=case["rope"],
                            io_dtype=case["io"], kv_dtype=case["kv"], prefix_len=prefix_len, cluster_sizes=sizes,
                            suffix_range=(case["suffix_lo"], case["suffix_hi"]), n_layers=case["layers"], seed=case["shape"])


class State:
    """A program's context, cache, plan and tensors; the library's objects go with it."""

    def __init__(self):
        self.ctx = self.cache = self.plan = None

    def __del__(self):
        if self.plan is not None:
            sgc.sgc_plan_destroy(self.plan)
        if self.cache is not None:
            sgc.sgc_cache_destroy(self.cache)
        if self.ctx is not None:
            sgc.sgc_ctx_destroy(self.ctx)


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _rows(t, cu):
    """Addresses of the row groups [cu[i], cu[i + 1]) of a packed tensor."""
    step = t.stride(0) * t.element_size()
    return [t.data_ptr() + int(a) * step for a in cu[:-1]]


def prepare(case, seed):
    w = _structure(case)
    s = State()
    s.case, s.w = case, w
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    io, L = TORCH[case["io"]], case["layers"]
    hq, hkv, d, T = case["hq"], case["hkv"], case["d"], w.total_suffix_tokens
    PT = int(w.prefix_len.sum())
    s.pcu = np.concatenate([[0], np.cumsum(w.prefix_len.astype(np.int64))])

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEVICE, dtype=io)

    # one channel per KV head, the same for prompts and questions
    chan = torch.randint(0, d, (hkv,), generator=g, device=DEVICE)

    def keys(n):
        k = normal(n, hkv, d)
        if case["outlier"] != 1.0:
            k[:, torch.arange(hkv, device=DEVICE), chan] *= case["outlier"]
        return k

    s.params = sgc.make_params(n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_layers=L, io_dtype=case["io"], kv_dtype=case["kv"],
                               rope_base=case["rope"], kernel=KERNELS[case["kernel"]],
                               max_position=int(w.prefix_len.max()) + int(w.suffix_len.max()) + case["steps"])
    s.ctx = sgc.sgc_ctx_create(s.params)
    pages = int(sum(-(-int(p) // 16) for p in w.prefix_len))
    nbytes = sgc.sgc_cache_pool_bytes(s.params, pages)
    s.pool = torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)
    s.cache = sgc.sgc_cache_create(s.ctx, s.pool.data_ptr(), nbytes, w.n_clusters)
    s.ids = list(range(w.n_clusters))
    s.lse = [torch.zeros((hq, T), device=DEVICE) if case["lse"] else None for _ in range(L)]

    if case["kind"] == "layer":
        dm, nq = case["d_model"], hq * d
        s.w_qkv = normal((hq + 2 * hkv) * d, dm) * (1.0 / math.sqrt(dm))
        s.w_o = normal(dm, nq) * (1.0 / math.sqrt(nq))
        s.px, s.x = normal(PT, dm), normal(T, dm)
        s.pq, s.q = (torch.empty((n, nq), dtype=io, device=DEVICE) for n in (PT, T))
        s.po, s.o = torch.empty_like(s.pq), torch.empty_like(s.q)
        s.py, s.y = torch.empty_like(s.px), torch.empty_like(s.x)
        s.px_rows, s.pq_rows, s.po_rows = (_rows(t, s.pcu) for t in (s.px, s.pq, s.po))
        _alloc(s)
        s.plan = _assign(s)
        sgc.sgc_plan_upload(s.ctx, s.plan, _stream())
        return s

    s.k, s.v = [keys(T) for _ in range(L)], [normal(T, hkv, d) for _ in range(L)]
    s.q = [normal(T, hq, d) for _ in range(L)]
    s.o = [torch.zeros_like(q) for q in s.q]
    if case["kind"] == "serve":
        s.pk, s.pv = [keys(PT) for _ in range(L)], [normal(PT, hkv, d) for _ in range(L)]
        s.pq = [normal(PT, hq, d) for _ in range(L)]
        s.po = [torch.zeros_like(q) for q in s.pq]
        s.prompt_rows = [tuple(_rows(t[layer], s.pcu) for t in (s.pq, s.pk, s.pv, s.po)) for layer in range(L)]
        return s

    # caches filled and plan made: what earlier calls of the program left behind
    _alloc(s)
    for layer in range(L):
        pk, pv = keys(PT), normal(PT, hkv, d)
        sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, s.ids, layer, None, _rows(pk, s.pcu), _rows(pv, s.pcu), None, None, _stream())
    s.plan = _assign(s)
    if case["kind"] == "decode":
        sgc.sgc_plan_enable_decode(s.ctx, s.plan, case["steps"])
        _suffix(s)
        n = w.n_queries
        s.tq, s.tk, s.tv = normal(case["steps"], n, hq, d), keys(case["steps"] * n).view(case["steps"], n, hkv, d), normal(case["steps"], n, hkv, d)
        s.to = torch.zeros_like(s.tq)
        s.tlse = torch.zeros((case["steps"], hq, n), device=DEVICE) if case["lse"] else None
    else:
        sgc.sgc_plan_upload(s.ctx, s.plan, _stream())
    return s


def _alloc(s):
    for c in s.ids:
        sgc.sgc_cache_alloc_cluster(s.ctx, s.cache, c, int(s.w.prefix_len[c]))


def _assign(s):
    return sgc.sgc_assign_clusters(s.ctx, s.cache, s.w.labels, s.w.suffix_len, s.w.n_clusters)[3]


def _suffix(s):
    for layer in range(s.case["layers"]):
        lse = s.lse[layer]
        sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, layer, s.q[layer].data_ptr(), s.k[layer].data_ptr(), s.v[layer].data_ptr(),
                                       s.o[layer].data_ptr(), None if lse is None else lse.data_ptr(), _stream())


def run(s):
    return {"serve": _serve, "suffix": _suffix_only, "decode": _decode, "layer": _layer}[s.case["kind"]](s)


def _outputs(s):
    return list(s.o) + [t for t in s.lse if t is not None]


def _serve(s):
    _alloc(s)
    for layer in range(s.case["layers"]):
        q, k, v, o = s.prompt_rows[layer]
        if len(s.ids) == 1:
            sgc.sgc_prefix_prefill(s.ctx, s.cache, 0, layer, q[0], k[0], v[0], o[0], None, int(s.w.prefix_len[0]), _stream())
        else:
            sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, s.ids, layer, q, k, v, o, None, _stream())
    s.plan = _assign(s)
    _suffix(s)
    sgc.sgc_plan_destroy(s.plan)
    s.plan = None
    for c in s.ids:             # one stream: whoever gets these pages next writes them behind the launches above
        sgc.sgc_cache_free_cluster(s.ctx, s.cache, c)
    return list(s.po) + _outputs(s)


def _suffix_only(s):
    _suffix(s)
    return _outputs(s)


def _decode(s):
    for step in range(s.case["steps"]):
        lse = None if s.tlse is None else s.tlse[step].data_ptr()
        sgc.sgc_decode_step_batched(s.ctx, s.cache, s.plan, 0, step, s.tq[step].data_ptr(), s.tk[step].data_ptr(), s.tv[step].data_ptr(),
                                    s.to[step].data_ptr(), lse, _stream())
    return [s.to] if s.tlse is None else [s.to, s.tlse]


def _layer(s):
    dm, st = s.case["d_model"], _stream()
    sgc.sgc_project_qkv_prefix_batched(s.ctx, s.cache, s.ids, 0, s.px_rows, s.w_qkv.data_ptr(), dm, s.pq_rows, st)
    sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, s.ids, 0, s.pq_rows, None, None, s.po_rows, None, st)
    sgc.sgc_project_out(s.ctx, s.po.data_ptr(), s.w_o.data_ptr(), dm, s.po.shape[0], s.py.data_ptr(), st)
    sgc.sgc_project_qkv_suffix(s.ctx, s.cache, s.plan, 0, s.x.data_ptr(), s.w_qkv.data_ptr(), dm, s.q.data_ptr(), st)
    sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, 0, s.q.data_ptr(), None, None, s.o.data_ptr(), None, st)
    sgc.sgc_project_out(s.ctx, s.o.data_ptr(), s.w_o.data_ptr(), dm, s.o.shape[0], s.y.data_ptr(), st)
    return [s.py, s.y]


def work(case):
    """Multiply-adds over visible keys (and of the projections); inputs once, outputs once.  Keys and values that a pass
    itself puts into pages are no input; a resident cache is one."""
    w = _structure(case)
    hq, hkv, d, L = case["hq"], case["hkv"], case["d"], case["layers"]
    P, S, T = w.prefix_len.astype(np.float64), w.suffix_len.astype(np.float64), float(w.total_suffix_tokens)
    PT, eb = float(P.sum()), w.io_bytes()
    prompt_flops = 2.0 * hq * d * float(np.sum(P * (P + 1.0)))
    row, kv_row = 2.0 * hq * d * eb, 2.0 * hkv * d * eb          # q in and o out; k and v in
    lse = 4.0 * hq * T if case["lse"] else 0.0
    cache = 2.0 * float(w.prefix_len[np.unique(w.labels)].sum()) * hkv * d * w.kv_bytes()
    if case["kind"] == "serve":
        return {"bytes": L * ((PT + T) * (row + kv_row) + lse), "flops": L * (prompt_flops + w.flops())}
    if case["kind"] == "suffix":
        return {"bytes": L * (cache + T * (row + kv_row) + lse), "flops": L * w.flops()}
    if case["kind"] == "decode":
        n, steps = float(w.n_queries), case["steps"]
        own = float(np.sum(S)) * steps + n * steps * (steps + 1) / 2.0       # own keys read over all steps
        lse = 4.0 * hq * n * steps if case["lse"] else 0.0
        return {"bytes": steps * (cache + n * (row + kv_row)) + own * 2.0 * hkv * d * eb + lse,
                "flops": 4.0 * hq * d * (steps * float(np.sum(P[w.labels])) + own)}
    dm, nq, nkv = case["d_model"], hq * d, hkv * d
    weights = float(dm) * (2 * nq + 2 * nkv) * eb
    return {"bytes": weights + (PT + T) * 2.0 * dm * eb,
            "flops": 2.0 * (PT + T) * dm * (2 * nq + 2 * nkv) + prompt_flops + w.flops()}


def tolerance(case):
    """About four times what a pass differs by from the same computation in 64 bits (2-norm): fp32 3e-7; 16-bit operands
    2.3e-3, with the projections around them 3.7e-3; fp8 caches 5e-3 (a key on a code boundary takes the other code when
    the rotation is summed differently, and a peaked row shows it), behind projections, whose keys are rounded to bf16
    first, 1.9e-2; query rows in e4m3 as well 2.8e-2."""
    if case["io"] == "f32":
        return {"rel": 1.5e-6}
    if case["kv"] == "fp8_e4m3":
        return {"rel": 0.03 if case["kernel"] == "mfma_fp8" or case["kind"] == "layer" else 0.02, "max": 0.9}
    return {"rel": 0.015 if case["kind"] == "layer" else 0.01}
