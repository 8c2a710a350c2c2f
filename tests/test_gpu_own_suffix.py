"""The question tokens' own keys in the matrix-core kernel, by each way they can reach it: as the caller gives them, out of suffix
pages (a plan with decode steps; its spare pages lie between the queries), and out of pages because an output overlaps the values.
Sizes around a page of 16 tokens, a chunk of four pages and a wavefront's 32 rows; tiles that touch one, four and more queries."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session, to_device, to_host_f32  # noqa: E402
from ref_util import fp8_query_floor, oracle_caches, oracle_suffix, tight_bar  # noqa: E402

SHAPES = [
    # head groups of 4: rows of one query, of four, of five in a tile
    (8, 2, [16], [33]), (8, 2, [70], [16, 15, 1, 17]), (8, 2, [64], [7, 6, 8, 5, 9, 1]),
    # more than one chunk of pages behind a tile; no cached keys
    (8, 1, [100], [63, 64, 65, 129]), (8, 2, [0, 1], [64, 1, 80, 16]),
    # no head groups: 128 tokens to a tile, many pages each
    (2, 2, [200, 40], [96, 24, 50, 31, 33, 128, 1, 1]), (1, 1, [65], [1] * 70),
]


def _run(w, route, kernel):
    with Session(w, kernel=kernel) as s:
        for c in range(w.n_clusters):
            s.alloc_cluster(c)
            s.prefix_prefill(c)
        s.assign()
        if route == "decode plan":
            s.enable_decode(20)
        dq, dk, dv = (to_device(x, "bf16") for x in w.suffix_qkv())
        dlse = torch.zeros((w.n_q_heads, dq.shape[0]), device="cuda:0")
        do = s.suffix_prefill(dq, dk, dv, do=dv if route == "output over the values" else None, dlse=dlse)
        torch.cuda.synchronize()
        return to_host_f32(do), dlse.cpu().numpy()


@pytest.mark.parametrize("kv,rope", [("bf16", 10000.0), ("bf16", 0.0), ("fp8_e4m3", 10000.0)])
@pytest.mark.parametrize("hq,hkv,prefix,suffix", SHAPES)
def test_own_keys_by_every_route(hq, hkv, prefix, suffix, kv, rope):
    labels = np.arange(len(suffix)) % len(prefix)
    w = workloads.custom("own", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=rope, io_dtype="bf16", kv_dtype=kv,
                         prefix_len=prefix, labels=labels.astype(np.int32), suffix_len=np.array(suffix, np.int32), seed=len(suffix))
    caches = oracle_caches(w)
    ref, lse = orc.suffix_prefill_batched(w.labels, w.cu_seqlens, [caches[c][0] for c in range(w.n_clusters)],
                                          [caches[c][1] for c in range(w.n_clusters)], *w.suffix_qkv(), w.rope_base)
    # 16-bit caches: four times an ideal 16-bit kernel's error; fp8: the bar the other tests use (a key on a code's boundary)
    bar, lse_bar = tight_bar(w, range(w.n_queries)) if kv == "bf16" else (6e-2, 2e-2)
    routes = ["as given", "decode plan"] + (["output over the values"] if hq == hkv else [])
    for route in routes:
        o, got_lse = _run(w, route, sgc.SGC_KERNEL_MFMA)
        assert float(np.abs(o - ref).max()) <= bar, route
        assert float(np.abs(got_lse - lse).max()) <= max(lse_bar, 2e-2), route
        if kv == "fp8_e4m3":        # query rows in e4m3 against the cache, in binary16 against own keys
            floor = max(fp8_query_floor(*caches[int(w.labels[n])], *w.suffix_qkv_query(n), w.rope_base) for n in range(w.n_queries) if prefix[labels[n]] > 0)
            o, _ = _run(w, route, sgc.SGC_KERNEL_MFMA_FP8)
            assert float(np.abs(o - ref).max()) <= 4 * floor + 6e-2, route


@pytest.mark.parametrize("hq,hkv,suffix", [(2, 1, [16, 16]), (4, 2, [8, 32, 8, 8, 16, 40]), (1, 1, [32, 32, 7]), (8, 1, [4, 4, 4, 20])])
def test_a_wavefront_sees_no_values_of_queries_it_has_no_rows_of(hq, hkv, suffix):
    """Values that are not finite may reach rows that share a wavefront's 32 with the query that has them, and no others."""
    g = hq // hkv
    w = workloads.custom("nan", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[40],
                         labels=np.zeros(len(suffix), np.int32), suffix_len=np.array(suffix, np.int32), seed=hq)
    cu = w.cu_seqlens
    with Session(w, kernel=sgc.SGC_KERNEL_MFMA) as s:
        s.alloc_cluster(0)
        s.prefix_prefill(0)
        s.assign()
        dq, dk, dv = (to_device(x, "bf16") for x in w.suffix_qkv())
        clean = to_host_f32(s.suffix_prefill(dq, dk, dv))
        for n in range(w.n_queries):
            bad = dv.clone()
            bad[cu[n]:cu[n + 1]] = float("nan")
            o = to_host_f32(s.suffix_prefill(dq, dk, bad))
            first, last = int(cu[n]) * g // 32, (int(cu[n + 1]) * g - 1) // 32      # wavefronts that hold rows of query n
            others = np.array([t for t in range(int(cu[-1])) if all(not first <= r // 32 <= last for r in range(t * g, t * g + g))], int)
            assert np.array_equal(o[others], clean[others]), n


@pytest.mark.parametrize("kv,kernel", [("bf16", sgc.SGC_KERNEL_MFMA), ("fp8_e4m3", sgc.SGC_KERNEL_MFMA), ("fp8_e4m3", sgc.SGC_KERNEL_MFMA_FP8)])
@pytest.mark.parametrize("hq,hkv,prefix,suffix", SHAPES)
def test_rows_as_given_and_pages_agree_bit_for_bit(hq, hkv, prefix, suffix, kv, kernel):
    """Both routes round an own key alike and walk the same pages."""
    w = workloads.custom("own_bits", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", kv_dtype=kv, prefix_len=prefix,
                         labels=(np.arange(len(suffix)) % len(prefix)).astype(np.int32), suffix_len=np.array(suffix, np.int32), seed=3)
    (o, lse), (op, lsep) = _run(w, "as given", kernel), _run(w, "decode plan", kernel)
    assert bool((o == op).all()) and bool((lse == lsep).all())


@pytest.mark.parametrize("hq,hkv,n,S", [(8, 1, 1, 256), (8, 1, 1, 257), (32, 8, 1, 900), (64, 8, 10, 112), (64, 8, 10, 113), (4, 4, 2, 1000), (8, 8, 18, 500)])
def test_long_questions_on_both_sides_of_the_rule(hq, hkv, n, S):
    """Own keys as rows where fewer than 4.5 tiles read a page (small launches: up to 16 pages), through pages above."""
    w = workloads.custom("long", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[40],
                         labels=np.zeros(n, np.int32), suffix_len=np.array([S] * n, np.int32), seed=S)
    o, lse = _run(w, "as given", sgc.SGC_KERNEL_MFMA)
    op, lsep = _run(w, "decode plan", sgc.SGC_KERNEL_MFMA)
    assert bool((o == op).all()) and bool((lse == lsep).all())
    some = [0, n - 1]
    rows, ref, ref_lse = oracle_suffix(w, queries=sorted(set(some)))
    bar, lse_bar = tight_bar(w, [0])
    assert float(np.abs(o[rows] - ref).max()) <= bar and float(np.abs(lse[:, rows] - ref_lse).max()) <= max(lse_bar, 2e-2)
