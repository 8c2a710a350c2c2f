"""The generic (fp32 matrix-core) attention kernel where its pieces begin and end: rows around its tiles of 16, prompts
around its blocks of 16 keys and around a turn of its wavefronts, tiles that hold several queries, empty prompts, head groups."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session, run_workload  # noqa: E402


@pytest.mark.parametrize("io,d,Hq,Hkv", [("f32", 64, 3, 1), ("f32", 128, 2, 2), ("bf16", 64, 4, 2)])
@pytest.mark.parametrize("prefix,suffix", [([0, 1], [1, 3]), ([15, 16], [16, 1]), ([17, 129], [5, 17]), ([64, 513], [40, 2])])
def test_generic_kernel_edges(io, d, Hq, Hkv, prefix, suffix):
    w = workloads.custom("generic", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, rope_base=10000.0, io_dtype=io, prefix_len=prefix,
                         cluster_sizes=[4, 3], suffix_range=(min(suffix), max(suffix)), seed=d + prefix[1])
    out = run_workload(w, kernel=sgc.SGC_KERNEL_GENERIC)
    caches = [orc.prefix_prefill(None, *w.prefix_kv(c), w.rope_base)[:2] for c in range(w.n_clusters)]
    o_ref, lse_ref = orc.suffix_prefill_batched(w.labels, w.cu_seqlens, [c[0] for c in caches], [c[1] for c in caches], *w.suffix_qkv(), w.rope_base)
    # fp32 throughout: sums of up to 128 products and 553 weights; bf16: one rounding of o (2^-9) on top of keys kept as binary16
    bar = 2e-5 if io == "f32" else 2e-2
    assert float(np.abs(out["o"] - o_ref).max()) <= bar
    assert float(np.abs(out["lse"] - lse_ref).max()) <= (2e-5 if io == "f32" else 2e-2)
    with Session(w, kernel=sgc.SGC_KERNEL_GENERIC) as s:        # the prompts' own causal attention, all in one launch
        for c in range(w.n_clusters):
            s.alloc_cluster(c)
        for c, (o, lse) in enumerate(s.prefix_prefill_batched(range(w.n_clusters), with_q=True, want_lse=True)):
            if w.prefix_len[c] == 0:
                continue
            _, _, po, pl = orc.prefix_prefill(w.prefix_q(c), *w.prefix_kv(c), w.rope_base, want_lse=True)
            assert float(np.abs(o.float().cpu().numpy() - po).max()) <= bar
            assert float(np.abs(lse.cpu().numpy() - pl).max()) <= bar


@pytest.mark.parametrize("io,kv,d", [("f32", "f32", 64), ("f32", "f32", 128), ("bf16", "bf16", 64), ("bf16", "fp8_e4m3", 64)])
def test_values_that_are_not_finite_stay_with_the_rows_that_see_them(io, kv, d):
    """Inf and NaN in a late prompt token's and in one query's K, V: rows that do not see the token are bit for bit those of
    the run with finite values, rows that see a value lose that one channel, rows that see a NaN key lose all."""
    Hq, Hkv = 4, 2
    w = workloads.custom("not_finite", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, rope_base=10000.0, io_dtype=io, kv_dtype=kv,
                         prefix_len=[40, 5], labels=[0, 0, 1, 0, 0], suffix_len=[5, 3, 2, 37, 4], seed=d)
    nan, inf = float("nan"), float("inf")

    def check(out, ref, first, heads, channel):
        """first[r]: row r sees the token; channel: the one that is lost, None for all"""
        for h in range(Hq):
            for r in range(ref.shape[0]):
                hit = bool(first[r]) and h in heads
                lost = np.zeros(d, bool)
                if hit:
                    lost[slice(None) if channel is None else channel] = True
                assert np.array_equal(np.isfinite(out[r, h]), ~lost), (r, h)
                assert np.array_equal(out[r, h][~lost], ref[r, h][~lost]), (r, h)

    def prompt(poison):
        with Session(w, kernel=sgc.SGC_KERNEL_GENERIC) as s:
            s.alloc_cluster(0)
            k, v = w.prefix_kv(0)
            poison(k, v)
            return s.prefix_prefill(0, k=k, v=v, with_q=True)[0].float().cpu().numpy()

    def batch(poison):
        with Session(w, kernel=sgc.SGC_KERNEL_GENERIC) as s:
            for c in range(2):
                s.alloc_cluster(c)
                s.prefix_prefill(c)
            s.assign()
            q, k, v = w.suffix_qkv()
            poison(k, v)
            o = s.suffix_prefill(*(torch.from_numpy(x).to(device="cuda:0", dtype=torch.float32 if io == "f32" else torch.bfloat16) for x in (q, k, v)))
            torch.cuda.synchronize()
            return o.float().cpu().numpy()

    group = {0: (0, 1), 1: (2, 3)}                      # KV head -> its query heads
    cu = np.asarray(w.cu_seqlens)
    query = np.searchsorted(cu, np.arange(cu[-1]), side="right") - 1
    clean_p, clean_b = prompt(lambda k, v: None), batch(lambda k, v: None)
    for hk, t, c, x in [(0, 35, 0, nan), (1, 39, d - 1, inf), (1, 16, 17, -inf), (0, 0, 3, nan)]:
        if kv != "fp8_e4m3" or x != x:                  # (an infinity would move the head's scale)
            def one(k, v):
                v[t, hk, c] = x
            check(prompt(one), clean_p, np.arange(40) >= t, group[hk], c)
        def key(k, v):
            k[t, hk, c] = nan
        check(prompt(key), clean_p, np.arange(40) >= t, group[hk], None)
    for hk, n, t, c, x in [(0, 0, 0, 0, inf), (1, 1, 2, d - 1, nan), (0, 3, 20, 5, -inf), (1, 3, 36, 33, nan), (0, 4, 1, 8, nan)]:
        sees = (query == n) & (np.arange(cu[-1]) >= cu[n] + t)
        def one(k, v):
            v[cu[n] + t, hk, c] = x
        check(batch(one), clean_b, sees, group[hk], c)
        def key(k, v):
            k[cu[n] + t, hk, c] = nan
        check(batch(key), clean_b, sees, group[hk], None)


@pytest.mark.parametrize("d,P,Hkv", [(64, 6001, 2), (128, 3000, 1)])
def test_fp32_sums_over_a_long_prompt(d, P, Hkv):
    """Error (2-norm) of rows over thousands of keys.  A chain of n additions of terms of random sign is off by about
    2^-24 sqrt(n / 6) of its result: 6.6e-7 for one chain through the 750 keys a wavefront has here; 1e-7 for 16 keys and
    1.7e-7 for the 47 blocks they come in.  Scores (two chains of d / 2 products) add 1.4e-7 to 2e-7, the exponentials and
    the normaliser 1e-7: 2.7e-7 to 3e-7 in all, and the bar is between that and the one chain."""
    w = workloads.custom("long_f32", n_q_heads=4, n_kv_heads=Hkv, head_dim=d, rope_base=500000.0, io_dtype="f32", prefix_len=[P],
                         cluster_sizes=[4], suffix_range=(33, 33), seed=d)
    out = run_workload(w, kernel=sgc.SGC_KERNEL_GENERIC)
    ck, cv = orc.prefix_prefill(None, *w.prefix_kv(0), w.rope_base)[:2]
    o_ref, _ = orc.suffix_prefill_batched(w.labels, w.cu_seqlens, [ck], [cv], *w.suffix_qkv(), w.rope_base)
    err = float(np.linalg.norm(out["o"] - o_ref) / np.linalg.norm(o_ref))
    print(f"d {d}, {P} keys: {err:.2e}", flush=True)
    assert err <= 4.2e-7
