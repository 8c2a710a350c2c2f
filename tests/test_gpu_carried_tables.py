"""Small calls whose tables travel with the launches: the same bits as the calls that copy their tables to the device first, at the
edges of what a launch's arguments hold (6 clusters; prompts: 480 pages, 256 tiles; questions: 144 pages of prompts, 40 own pages,
48 queries, 40 tiles, 4 queries a tile; generic kernel: 240 pages, 160 tiles, 64 queries) and just past them, where both sides copy.  Each
case says which of its two calls carries its tables, and the library has to agree."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_10951_amd import sgc, workloads
from paper_2505_10951_amd.harness import Session, to_device

pytestmark = pytest.mark.gpu


def _pass(w, copied):
    """Whether the prompts' and the batch's tables were carried; prompts' outputs and LSE, the batch's outputs and LSE.  copied: every table
    goes through the device's copies."""
    with Session(w) as s:
        carried = lambda: sgc.lib().sgc_debug_carried(s.ctx) == 1
        for c in range(w.n_clusters):
            s.alloc_cluster(c)
        if copied:
            s.assign()
            s.enable_decode(1)
        prompts = s.prefix_prefill_batched(list(range(w.n_clusters)), 0, with_q=True, want_lse=True)
        routes = [carried()]
        s.assign()
        if copied:
            s.upload_plan()
        lse = torch.zeros((w.n_q_heads, w.total_suffix_tokens), device="cuda:0")
        o = s.suffix_prefill(*(to_device(x, "bf16") for x in w.suffix_qkv()), dlse=lse)
        routes.append(carried())
        again = s.suffix_prefill(*(to_device(x, "bf16") for x in w.suffix_qkv()))
        torch.cuda.synchronize()
        assert torch.equal(o, again)
        return routes, [t.clone() for pair in prompts for t in pair if t is not None and t.numel()] + [o.clone(), lse]


@pytest.mark.parametrize("hq,hkv,prefix,sizes,suffix,prompts,batch", [
    (32, 8, [411], [1], (23, 23), True, True),
    (8, 2, [1, 16, 17, 0, 200, 64], [1, 2, 1, 3, 1, 1], (1, 30), True, True),
    (8, 2, [5, 9, 30, 1, 64, 65, 66], [1] * 7, (1, 9), False, False),       # seven clusters
    (2, 2, [2304], [2], (30, 40), True, True), (2, 2, [2305], [2], (30, 40), True, False),      # 144 pages of prompts, 145
    (4, 4, [3840, 3840], [1, 0], (3, 3), True, False), (4, 4, [3840, 3841], [1, 0], (3, 3), False, False),      # 480 pages, 481
    (2, 2, [7680], [1], (3, 3), False, False),                              # 120 tiles, but 60 on one XCD: 480 with padding
    (32, 8, [1024], [1], (9, 9), True, True), (32, 8, [1025], [1], (9, 9), False, True),        # 256 tiles, 264
    (8, 8, [100], [48], (5, 8), True, False), (32, 8, [70], [40], (1, 2), True, False),         # more than four queries a tile
    (2, 2, [70], [10], [49] * 10, True, True), (2, 2, [70], [11], [49] * 10 + [16], True, False),       # 40 own pages, 41
    (2, 2, [70, 5], [10, 38], [49] * 10 + [0] * 38, True, True), (2, 2, [70, 5], [10, 39], [49] * 10 + [0] * 39, True, False),  # 48 queries, 49, most without tokens
    (32, 8, [300], [10], (16, 16), True, True), (32, 8, [300], [11], (16, 16), True, False),    # five tiles a KV head, six
])
def test_same_bits_as_copied_tables(hq, hkv, prefix, sizes, suffix, prompts, batch):
    lens = {"suffix_range": suffix, "cluster_sizes": sizes} if isinstance(suffix, tuple) else {"suffix_len": suffix, "labels": np.repeat(np.arange(len(sizes)), sizes)}
    w = workloads.custom("carried", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=500000.0, io_dtype="bf16", prefix_len=prefix,
                         seed=len(prefix) + sum(sizes), **lens)
    (routes, got), (copied, ref) = _pass(w, False), _pass(w, True)
    assert routes == [prompts, batch] and copied == [False, False]
    for a, b in zip(got, ref):
        assert torch.isfinite(a).all() and torch.equal(a, b)


def test_captured_calls_and_calls_that_copy_behind_them():
    """Replays take the tables of the calls that were captured; a batch that is too large behind a prompt whose tables were carried
    brings the page tables to the device itself."""
    w = workloads.custom("carried_graph", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[300, 90],
                         cluster_sizes=[2, 3], suffix_range=(4, 20), seed=3)
    big = workloads.custom("carried_big", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[300, 90],
                           cluster_sizes=[60, 40], suffix_range=(4, 20), seed=4)
    with Session(w) as s:
        for c in range(2):
            s.alloc_cluster(c)
        s.prefix_prefill_batched([0, 1], 0, with_q=True)
        s.assign()
        q, k, v = (to_device(x, "bf16") for x in w.suffix_qkv())
        o = torch.empty_like(q)
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            s.suffix_prefill(q, k, v, do=o)
        side.synchronize()
        first = o.clone()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            s.suffix_prefill(q, k, v, do=o)
        for step in range(3):
            q.copy_(to_device(w.suffix_qkv()[0], "bf16") * (1.0 + step))
            o.zero_()
            g.replay()
            torch.cuda.synchronize()
            eager = s.suffix_prefill(q, k, v)
            torch.cuda.synchronize()
            assert torch.equal(o, eager) and (step > 0 or torch.equal(o, first))
        bq, bk, bv = (to_device(x, "bf16") for x in big.suffix_qkv())
        s.assign(big.labels, big.suffix_len)
        got = s.suffix_prefill(bq, bk, bv).clone()
        s.upload_plan()
        s.assign(big.labels, big.suffix_len)
        s.upload_plan()
        assert torch.equal(got, s.suffix_prefill(bq, bk, bv))
        torch.cuda.synchronize()


@pytest.mark.parametrize("io,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("hq,hkv,prefix,sizes,suffix,prompts_carried,batch_carried", [
    (4, 4, [192, 256], [8, 8], (16, 32), True, True),
    (8, 2, [1, 16, 0, 17, 200, 64], [1, 2, 1, 3, 1, 1], (1, 30), True, True),
    (4, 2, [300], [64], (1, 9), True, True), (4, 2, [300], [65], (1, 9), True, False),         # 64 queries, 65
    (4, 1, [640], [1], (640, 640), True, True), (4, 1, [641], [1], (641, 641), False, False),   # 160 tiles, 161
    (1, 1, [2560, 1280], [1, 1], (9, 9), False, True), (1, 1, [2560, 1281], [1, 1], (9, 9), False, False),      # 240 pages, 241; 240 tiles
    (2, 2, [1920, 640], [1, 1], (9, 9), True, True), (2, 2, [1920, 641], [1, 1], (9, 9), False, True),          # 160 tiles of prompts, 161
    (16, 16, [40, 7, 1], [5, 20, 0], (0, 4), True, True),                                      # queries without tokens, many in a tile
])
def test_generic_kernel_same_bits_as_copied_tables(io, d, hq, hkv, prefix, sizes, suffix, prompts_carried, batch_carried):
    """Prompts: alone against in a call with a prompt of 300 pages, which copies its tables; batch: against an uploaded plan."""
    w = workloads.custom("carried_generic", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rope_base=10000.0, io_dtype=io, kv_dtype=io,
                         prefix_len=prefix + [4800], cluster_sizes=sizes + [0], suffix_range=suffix, seed=len(prefix) + sum(sizes))
    n = len(prefix)
    out = []
    for copied in (False, True):
        with Session(w) as s:
            carried = lambda: sgc.lib().sgc_debug_carried(s.ctx) == 1
            for c in range(n + 1):
                s.alloc_cluster(c)
            prompts = s.prefix_prefill_batched(list(range(n + 1 if copied else n)), 0, with_q=True, want_lse=True)[:n]
            assert carried() == (prompts_carried and not copied)
            s.assign()
            if copied:
                s.upload_plan()
            lse = torch.zeros((hq, w.total_suffix_tokens), device="cuda:0")
            o = s.suffix_prefill(*(to_device(x, io) for x in w.suffix_qkv()), dlse=lse)
            torch.cuda.synchronize()
            assert carried() == (batch_carried and not copied)
            out.append([t.clone() for pair in prompts for t in pair if t.numel()] + [o.clone(), lse])
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("layers", [1, 6, 7, 32])
def test_contexts_of_many_layers_copy(layers):
    """Where many layers follow each other tables in the launch's arguments are the slower: they are copied, for prompts and batch."""
    w = workloads.custom("carried_layers", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[100],
                         cluster_sizes=[2], suffix_range=(5, 9), n_layers=layers, seed=layers)
    with Session(w) as s:
        s.alloc_cluster(0)
        s.prefix_prefill_batched([0], layers - 1, with_q=True)
        assert sgc.lib().sgc_debug_carried(s.ctx) == (layers <= 6)
        s.assign()
        s.suffix_prefill(*(to_device(x, "bf16") for x in w.suffix_qkv(layers - 1)), layer=layers - 1)
        torch.cuda.synchronize()
        assert sgc.lib().sgc_debug_carried(s.ctx) == (layers <= 6)


def test_prompts_around_decode_steps():
    """A program that serves batch after batch and generates: prompts' tables are carried before a batch has decode steps and again once its plan
    is gone, not while it is there; and the steps, those that may not allocate among them, find the page tables that they need."""
    w = workloads.custom("carried_decode", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[300, 90, 40],
                         cluster_sizes=[2, 3, 0], suffix_range=(4, 20), seed=3)
    q, k, v = (to_device(x, "bf16") for x in w.suffix_qkv())
    steps = [tuple(to_device(x, "bf16") for x in w.decode_qkv(t)) for t in range(2)]
    results = []
    with Session(w) as s:
        carried = lambda: sgc.lib().sgc_debug_carried(s.ctx) == 1
        for batch in range(3):
            for c in (0, 1) if batch % 2 == 0 else (1, 0):           # other pages the second time
                s.alloc_cluster(c)
            s.prefix_prefill_batched([0, 1], 0, with_q=True)
            assert carried()
            s.assign()
            s.enable_decode(2)
            s.suffix_prefill(q, k, v)
            got = []
            for t, (dq, dk, dv) in enumerate(steps):
                o = torch.empty_like(dq)
                entry = sgc.sgc_decode_step_batched_noalloc if batch else sgc.sgc_decode_step_batched
                entry(s.ctx, s.cache, s.plan, 0, t, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), o.data_ptr(), None, s.stream)
                got.append(o)
            s.alloc_cluster(2)
            s.prefix_prefill_batched([2], 0, with_q=True)
            assert not carried()
            s.decode_step(1, *steps[1], do=got[1])
            torch.cuda.synchronize()
            results.append(torch.stack(got))
            sgc.sgc_plan_destroy(s.plan)
            s.plan = None
            for c in range(3):
                s.free_cluster(c)
    assert all(torch.isfinite(r).all() and torch.equal(r, results[0]) for r in results)


def test_a_plan_used_again_is_uploaded():
    """Six calls on a plan carry their tables, the seventh uploads it: the same bits, also where clusters came and went in between."""
    w = workloads.custom("carried_again", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[100, 70, 33],
                         cluster_sizes=[2, 1, 0], suffix_range=(5, 40), seed=2)
    q, k, v = (to_device(x, "bf16") for x in w.suffix_qkv())
    with Session(w) as s:
        for c in range(2):
            s.alloc_cluster(c)
        s.prefix_prefill_batched([0, 1], 0)
        s.assign()
        first = s.suffix_prefill(q, k, v).clone()
        for call in range(2, 11):
            if call == 8:
                s.alloc_cluster(2)
            assert torch.equal(s.suffix_prefill(q, k, v), first)
            assert sgc.lib().sgc_debug_carried(s.ctx) == (call <= 6)
        torch.cuda.synchronize()


@pytest.mark.parametrize("layers", [1, 32])
def test_captured_calls_carry(layers):
    """A captured call's tables go with it in contexts of many layers too, and on a plan that has carried them six times: copies would need a
    staging buffer and memory while the stream is being captured."""
    w = workloads.custom("carried_captured", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[100, 70],
                         cluster_sizes=[2, 1], suffix_range=(5, 40), n_layers=layers, seed=4)
    q, k, v = (to_device(x, "bf16") for x in w.suffix_qkv())
    with Session(w) as s:
        for c in range(2):
            s.alloc_cluster(c)
        prompts = s.prefix_prefill_batched([0, 1], 0, with_q=True)
        s.assign()
        g = torch.cuda.CUDAGraph()
        o = torch.empty_like(q)
        pq, (pk, pv) = to_device(w.prefix_q(1), "bf16"), (to_device(x, "bf16") for x in w.prefix_kv(1))
        po = torch.empty_like(pq)
        if layers == 1:
            for _ in range(6):
                s.suffix_prefill(q, k, v, do=o)
        with torch.cuda.graph(g):
            stream = torch.cuda.current_stream().cuda_stream
            sgc.sgc_prefix_prefill(s.ctx, s.cache, 1, 0, pq.data_ptr(), pk.data_ptr(), pv.data_ptr(), po.data_ptr(), None, 70, stream)
            assert sgc.lib().sgc_debug_carried(s.ctx) == 1
            sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, 0, q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), None, stream)
        assert sgc.lib().sgc_debug_carried(s.ctx) == 1
        for _ in range(3):
            o.zero_()
            po.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, s.suffix_prefill(q, k, v)) and torch.equal(po, prompts[1][0])
            assert sgc.lib().sgc_debug_carried(s.ctx) == 0
