"""Decode steps of few rows, one launch: a workgroup has one group of 32 rows and one key range, its eight wavefronts share cached and own
keys, and the last range of a row tile adds up.  Sizes around a wavefront's 32 keys, a page of 16 and the eight wavefronts' 256; up
to 32 rows of a cluster and KV head and, in two launches, above that; the limits of the rule that says where it is taken, from both sides
(tests/test_decode_plan.py has the rule itself)."""
import numpy as np
import pytest

pytest.importorskip("torch")

from paper_2505_10951_amd import workloads
from ref_util import oracle_caches
from test_decode_plan import decode_plan
from test_gpu_decode import TOL, _oracle_decode, _run_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix", [[1, 15], [31, 33], [64, 65], [66, 1], [97, 95], [255, 256], [257, 300], [2000, 1]])
@pytest.mark.parametrize("hq,hkv,per", [(8, 2, 1), (8, 2, 8), (8, 2, 9), (8, 1, 4), (32, 32, 3), (160, 80, 16)])
def test_rows_and_keys_around_a_wavefront(hq, hkv, per, prefix):
    """(80 heads of two clusters: 160 row tiles)"""
    w = workloads.custom("few", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=500000.0, io_dtype="bf16", prefix_len=prefix,
                         cluster_sizes=[per, per], suffix_range=(1, 20), seed=per, k_outlier_scale=8.0 if prefix[0] == 2000 else 1.0)
    o, lse = _run_decode(w, 2)[0]
    o_ref, lse_ref = _oracle_decode(w, 0, 2, oracle_caches(w, 0))
    assert np.isfinite(o).all() and np.abs(o - o_ref).max() <= TOL["bf16"] and np.abs(lse - lse_ref).max() <= 5e-2


@pytest.mark.parametrize("prefix,masked", [(40, (0, 32)), (300, (32, 64)), (300, (0, 256)), (900, (640, 899))])
def test_keys_that_score_minus_infinity(prefix, masked):
    """Whole units of 32 keys with scores of minus infinity count for nothing; the other keys' result stays."""
    import torch
    from oracle import oracle as orc
    from paper_2505_10951_amd.harness import Session, to_device, to_host_f32
    w = workloads.custom("few_inf", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=0.0, io_dtype="bf16", prefix_len=[prefix],
                         cluster_sizes=[3], suffix_range=(2, 5), seed=prefix)
    pk, pv = w.prefix_kv(0)
    pk = pk.copy()
    pk[masked[0]:masked[1], :, 5] = -np.inf
    with Session(w) as s:
        s.alloc_cluster(0)
        s.prefix_prefill(0, k=pk, v=pv)
        s.assign()
        s.enable_decode(2)
        q, k, v = w.suffix_qkv()
        q[:, :, 5] = np.abs(q[:, :, 5])
        s.suffix_prefill(*(to_device(x, "bf16") for x in (q, k, v)))
        dq, dk, dv = w.decode_qkv(0)
        dq[:, :, 5] = np.abs(dq[:, :, 5])
        lse = torch.zeros((8, 3), device="cuda:0")
        o = s.decode_step(0, *(to_device(x, "bf16") for x in (dq, dk, dv)), dlse=lse)
        torch.cuda.synchronize()
        o, lse = to_host_f32(o), lse.cpu().numpy()
    keep = np.r_[0:masked[0], masked[1]:prefix]
    cu = w.cu_seqlens
    for n in range(3):
        a, b = int(cu[n]), int(cu[n + 1])
        S = b - a
        ref, ref_lse, _ = orc.suffix_prefill(pk[keep], pv[keep], np.concatenate([q[a:b], dq[n:n + 1]]), np.concatenate([k[a:b], dk[n:n + 1]]),
                                             np.concatenate([v[a:b], dv[n:n + 1]]), 0.0)
        assert np.abs(o[n] - ref[S]).max() <= TOL["bf16"] and np.abs(lse[:, n] - ref_lse[:, S]).max() <= 5e-2


@pytest.mark.parametrize("hq,hkv,per,prefix,suffix", [(32, 1, 1, [700], (1, 40)),          # 32 heads: two tasks of 16 for a query's own keys
                                                       (20, 1, 1, [64, 0], (3, 60)),        # 20 heads: a task that is not full
                                                       (4, 1, 8, [1500], (90, 300)),        # long questions: more tasks than one range has wavefronts
                                                       (2, 2, 32, [5, 0], (1, 33)),         # 32 queries a row tile, hardly any cached keys
                                                       (8, 2, 3, [4000, 100], (16, 16))])   # many ranges, one cluster far shorter
def test_own_keys_of_a_step(hq, hkv, per, prefix, suffix):
    """18 steps (the new tokens cross a page boundary), the queries' own keys in the launch of the cached ones."""
    w = workloads.custom("few_own", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=prefix,
                         cluster_sizes=[per] * len(prefix), suffix_range=suffix, seed=hq + per)
    o, lse = _run_decode(w, 18)[0]
    o_ref, lse_ref = _oracle_decode(w, 0, 18, oracle_caches(w, 0))
    assert np.isfinite(o).all() and np.abs(o - o_ref).max() <= TOL["bf16"] and np.abs(lse - lse_ref).max() <= 5e-2


@pytest.mark.parametrize("hq,hkv,sizes,prefix,suffix,one", [
    (8, 8, [28], [1100], (100, 140), True), (8, 2, [8], [900], (350, 500), True),       # many own keys
    (8, 8, [28], [60], (100, 140), False),                                              # ... over one 64-key step
    (16, 16, [16, 2, 1], [150, 150, 150], (90, 110), True), (32, 32, [31, 2, 1], [150, 150, 150], (90, 110), False),      # uneven clusters
    (32, 32, [2] * 8, [300, 40] * 4, (1, 30), True),                                    # 256 row tiles, one range
    (8, 8, [14] + [1] * 32, [700] + [300] * 32, (1, 30), True), (8, 8, [15] + [1] * 32, [700] + [300] * 32, (1, 30), False),      # 264, of up to 14 rows and of 15
    (8, 8, [1] * 128, [900] * 128, (1, 30), True), (8, 8, [1] * 129, [900] * 129, (1, 30), False),     # 1024 row tiles, and past them
])
def test_limits_of_the_rule(hq, hkv, sizes, prefix, suffix, one):
    w = workloads.custom("few_limits", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=prefix,
                         cluster_sizes=sizes, suffix_range=suffix, seed=hq + sizes[0])
    assert decode_plan(hq, hkv, [(n, int(w.suffix_len[w.labels == c].mean()), P) for c, (n, P) in enumerate(zip(sizes, prefix))], steps=2)[0] == one
    o, lse = _run_decode(w, 2)[0]
    assert np.isfinite(o).all()
    some = np.unique(np.linspace(0, w.n_queries - 1, 40).astype(int))
    o_ref, lse_ref = _oracle_decode(w, 0, 2, oracle_caches(w, 0), queries=some)
    assert np.abs(o[:, some] - o_ref[:, some]).max() <= TOL["bf16"] and np.abs(lse[:, :, some] - lse_ref[:, :, some]).max() <= 5e-2


def test_step_again_overlapping_and_with_a_value_that_is_not_finite():
    """The same step twice gives the same bits (the ranges' counters are back at zero); an output that overlaps the new tokens, whose
    rows must not be stored before all are read, gives the same result within rounding; a NaN value of one query stays with it."""
    import torch
    from paper_2505_10951_amd import sgc
    from paper_2505_10951_amd.harness import Session, to_device, to_host_f32
    w = workloads.custom("few_again", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=500000.0, io_dtype="bf16", prefix_len=[3000, 40],
                         cluster_sizes=[4, 2], suffix_range=(2, 30), seed=5)
    with Session(w) as s:
        for c in range(2):
            s.alloc_cluster(c)
        s.prefix_prefill_batched([0, 1], 0)
        s.assign()
        s.enable_decode(2)
        s.suffix_prefill(*(to_device(x, "bf16") for x in w.suffix_qkv()))
        dq, dk, dv = (to_device(x, "bf16") for x in w.decode_qkv(0))
        first = s.decode_step(0, dq, dk, dv).clone()
        assert sgc.lib().sgc_debug_one_launch(s.ctx)
        for _ in range(3):
            assert torch.equal(s.decode_step(0, dq, dk, dv), first)
        n, hq, d = dq.shape
        both = torch.zeros(n * hq * d + dk.numel(), dtype=dq.dtype, device="cuda:0")
        o, k = both[:n * hq * d].view(n, hq, d), both[n * hq * d - dk.numel():n * hq * d].view(dk.shape)
        k.copy_(dk)
        s.decode_step(0, dq, k, dv, do=o)
        torch.cuda.synchronize()
        assert not sgc.lib().sgc_debug_one_launch(s.ctx)
        assert np.abs(to_host_f32(o) - to_host_f32(first)).max() <= 1e-2
        # outputs that end where the new keys begin do not overlap them: one launch, the same bits
        one = torch.zeros(n * hq * 2 + dk.numel(), dtype=dq.dtype, device="cuda:0")
        lse, k = one[:n * hq * 2].view(torch.float32).view(hq, n), one[n * hq * 2:].view(dk.shape)
        k.copy_(dk)
        assert torch.equal(s.decode_step(0, dq, k, dv, dlse=lse), first) and sgc.lib().sgc_debug_one_launch(s.ctx)
        bad = dv.clone()
        bad[1, 0, 7] = float("nan")
        o = to_host_f32(s.decode_step(0, dq, dk, bad))
        assert np.isnan(o[1, :4, 7]).all()
        o[1, :4, 7] = to_host_f32(first)[1, :4, 7]
        assert np.array_equal(o, to_host_f32(first))


@pytest.mark.parametrize("noalloc", [True, False])
def test_captured_steps(noalloc):
    """Replays of captured steps, with other steps between them, give the eager steps' bits, also where the counters of the array of callers
    that cannot allocate hold what later steps that ran into each other would leave there.  Steps captured on a plan that has run none (its
    block, counters included, is new) neither need that capture to be replayed nor leave the eager steps behind it without cleared counters."""
    import torch
    from paper_2505_10951_amd import sgc
    from paper_2505_10951_amd.harness import Session, to_device
    w = workloads.custom("few_graph", n_q_heads=8, n_kv_heads=2, head_dim=128, rope_base=500000.0, io_dtype="bf16", prefix_len=[2500, 700],
                         cluster_sizes=[3, 2], suffix_range=(2, 30), seed=9)
    call = sgc.sgc_decode_step_batched_noalloc if noalloc else sgc.sgc_decode_step_batched
    with Session(w) as s:
        for c in range(2):
            s.alloc_cluster(c)
        s.prefix_prefill_batched([0, 1], 0)
        s.assign()
        s.enable_decode(3)
        s.suffix_prefill(*(to_device(x, "bf16") for x in w.suffix_qkv()))
        steps = [tuple(to_device(x, "bf16") for x in w.decode_qkv(t)) for t in range(3)]
        outs = [torch.zeros_like(q) for q, _, _ in steps]

        def run(stream):
            for t, (q, k, v) in enumerate(steps):
                call(s.ctx, s.cache, s.plan, 0, t, q.data_ptr(), k.data_ptr(), v.data_ptr(), outs[t].data_ptr(), None, stream)

        def capture():
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                run(torch.cuda.current_stream().cuda_stream)
            return g

        def check(do):
            for o in outs:
                o.fill_(7.0)
            do()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(outs, ref))

        # the reference: another plan of the same batch, eager
        run(s.stream)
        torch.cuda.synchronize()
        ref = [o.clone() for o in outs]
        assert all(torch.isfinite(o).all() for o in ref)
        s.assign()
        s.enable_decode(3)
        s.suffix_prefill(*(to_device(x, "bf16") for x in w.suffix_qkv()))
        torch.cuda.synchronize()
        dropped = capture()
        check(lambda: run(s.stream))
        del dropped
        first, second = capture(), capture()
        for k in (0, 1, 2, 5):
            check(lambda: run(s.stream))
            if noalloc and k:
                sgc.lib().sgc_debug_leave_in_counters(s.ctx, k)
            check(second.replay)
            check(first.replay)
            check(first.replay)
        if noalloc:
            sgc.lib().sgc_debug_leave_in_counters(s.ctx, 1)
        check(lambda: run(s.stream))
