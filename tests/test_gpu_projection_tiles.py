"""The projections in every tile size the planner chooses from (256 x 256, 128 x 128 in two depths, 64 x 128, 64 x 64, and
256-row slabs with a remainder in smaller tiles), at rows where a tile begins, ends or is left nearly empty, against plain
fp32 products.

Error bar of y and q: the products are exact in fp32, a sum of K unit-variance terms scaled by 1/sqrt(K) is off by about
2^-24 sqrt(K) <= 4e-6 in any order, and the result is rounded to bf16 once: |err| <= 2^-9 |ref| + 2^-16, doubled here for
sums that the two orders put on different sides of a rounding boundary (a whole bf16 step is 2^-8 |ref|)."""
import numpy as np
import pytest

from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session, to_device  # noqa: E402
from test_gpu_layer import _run_layer  # noqa: E402
from test_projection_plan import PAGES, PLAIN, SLOTS, plan as tiles_of  # noqa: E402


def _close(name, got, ref):
    err = (got.float() - ref).abs()
    bar = 2.0 ** -8 * ref.abs() + 2.0 ** -15
    worst = float((err / bar).max())
    print(f"{name}: worst err/bar {worst:.3f}", flush=True)
    assert worst <= 1.0, name


# (rows, columns, heads of 128 = contraction / 128, choice of tiles as test_projection_plan numbers them)
@pytest.mark.parametrize("M,N,Hq,choice", [
    (1, 128, 4, 4), (64, 256, 3, 4), (129, 4096, 5, 4),                          # 64 x 64: fewer rows than a tile, odd ones
    (200, 4224, 7, 3), (300, 4096, 32, 3),                                       # 64 x 128
    (257, 8192, 4, 1), (600, 4096, 32, 1), (1000, 4096, 8, 1),                   # 128 x 128, deep
    (1, 128, 1, 2), (63, 128, 1, 2), (65, 384, 2, 2),                            # 128 x 128, two workgroups per CU: two and four
    (2000, 4096, 32, 2), (2048, 4096, 7, 2),                                     # steps, many, few in many tiles
    (16384, 4096, 1, 2), (16300, 4096, 2, 2), (16384, 4096, 3, 2),
    (4097, 2048, 1, 0), (4097, 2048, 2, 0), (4097, 2048, 3, 0),                  # 256 x 256: fewer steps than the ring of slabs
    (4096, 4096, 32, 0),
    (4300, 4224, 8, 11), (5000, 4224, 16, 12), (4095, 4224, 7, 13), (4300, 4096, 32, 14),     # 256 x 256 and a remainder
])
def test_output_projection_rows_and_tiles(M, N, Hq, choice):
    assert tiles_of([M], N, Hq * 128, 0, PLAIN)[0] == choice
    g = torch.Generator(device="cuda:0").manual_seed(M + N)
    K = Hq * 128
    x = torch.randn((M, K), generator=g, device="cuda:0", dtype=torch.bfloat16)
    w = torch.randn((N, K), generator=g, device="cuda:0", dtype=torch.bfloat16) * K ** -0.5
    y = torch.full((M + 1, N), 7.0, device="cuda:0", dtype=torch.bfloat16)
    ctx = sgc.sgc_ctx_create(sgc.make_params(n_q_heads=Hq, n_kv_heads=Hq, head_dim=128, io_dtype="bf16"))
    sgc.sgc_project_out(ctx, x.data_ptr(), w.data_ptr(), N, M, y.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    sgc.sgc_ctx_destroy(ctx)
    _close(f"{M} x {N} x {K}", y[:M], x.float() @ w.float().T)
    assert bool((y[M] == 7.0).all()), "a row behind the last was written"


@pytest.mark.parametrize("Hq,Hkv,d_model,rows", [(32, 8, 4096, 300), (16, 8, 1024, 1000), (16, 8, 1024, 2001), (2, 1, 64, 17)])
def test_qkv_epilogues_per_tile(Hq, Hkv, d_model, rows):
    """Queries, pages of the prompt and (through the attention over an empty prompt) pages of the batch."""
    prompt = workloads.custom("tiles", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16",
                              prefix_len=[rows, 0], cluster_sizes=[1, max(1, rows // 48)], suffix_range=(33, 64), seed=rows)
    last = prompt.n_queries - 1
    _run_layer(prompt, d_model, queries=sorted({0, last // 2, last}))


@pytest.mark.parametrize("Hq,Hkv,d_model,prompts,choice", [
    (2, 1, 64, [17], 4), (32, 32, 2048, [33, 32], 3), (32, 8, 256, [500], 1), (32, 32, 64, [129], 2), (16, 8, 1024, [2001], 2),
    (32, 8, 2048, [777, 300, 33], 0),
    # the cut falls inside a prompt; every cached row is compared
    (32, 32, 2048, [777, 367, 33], 11), (32, 32, 2048, [500, 1700, 700], 12), (32, 32, 2048, [367, 777, 33], 13), (32, 32, 1024, [500, 500, 300], 14),
])
def test_prompt_projection_in_every_tile(Hq, Hkv, d_model, prompts, choice):
    """Queries, keys and values of prompts: pages row by row, queries through the prompts' outputs."""
    n_kv = 2 * Hkv * 128
    got, n_slabs, big = tiles_of(prompts, Hq * 128 + n_kv, d_model, n_kv, PAGES)
    assert got == choice and (choice < 10 or 0 < big < n_slabs)
    w = workloads.custom("prompt_tiles", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16",
                         prefix_len=prompts, cluster_sizes=[1] * len(prompts), suffix_range=(3, 9), seed=d_model + choice)
    _run_layer(w, d_model)


@pytest.mark.parametrize("Hq,Hkv,d_model,T,choice", [
    (2, 1, 64, 17, 4), (32, 8, 4096, 129, 3), (4, 2, 4096, 3500, 1), (8, 8, 64, 4200, 2), (16, 8, 64, 3500, 0),
    (16, 8, 4096, 5000, 11), (32, 8, 4096, 3500, 12), (32, 32, 4096, 1400, 13), (32, 32, 1024, 1400, 14),
])
def test_batch_projection_in_every_tile(Hq, Hkv, d_model, T, choice):
    """Queries, keys and values of a batch, through the attention of questions that have no prompt: the first and the last of
    them, and those on both sides of the row where a second launch begins."""
    n_kv = 2 * Hkv * 128
    got, n_slabs, big = tiles_of([T], Hq * 128 + n_kv, d_model, n_kv, SLOTS)
    assert got == choice and (choice < 10 or 0 < big < n_slabs)
    lens = [41] * (T // 41) + [T % 41]
    w = workloads.custom("batch_tiles", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16",
                         prefix_len=[0], labels=[0] * len(lens), suffix_len=lens, seed=T)
    cut = (256 * big if 0 < big < n_slabs else T // 2) // 41
    _run_layer(w, d_model, queries=sorted({0, max(0, cut - 1), cut, min(cut + 1, len(lens) - 1), len(lens) - 1}))


def test_prompt_alone_and_among_others():
    """Which tiles a call takes depends on all of its rows, and tiles differ in the order of their fp32 sums (off by
    2^-24 sqrt(K) <= 4e-6 each): what a prompt leaves in its pages may differ by the rounding of the stored type, one step of
    bf16 (V) or binary16 (K), when it is projected by itself and among others; no more than that, and in few places."""
    Hq, Hkv, d_model, prompts = 32, 8, 4096, [300] + [1024] * 9
    n_kv = 2 * Hkv * 128
    assert tiles_of(prompts[:1], Hq * 128 + n_kv, d_model, n_kv, PAGES)[0] != tiles_of(prompts, Hq * 128 + n_kv, d_model, n_kv, PAGES)[0]
    w = workloads.custom("alone", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16",
                         prefix_len=prompts, cluster_sizes=[1] * 10, suffix_range=(3, 9), seed=3)
    dw, dwo = (to_device(x, "bf16") for x in w.layer_weights(d_model))
    got = []
    for clusters in ([0], list(range(10))):
        with Session(w) as s:
            for c in clusters:
                s.alloc_cluster(c)
            s.layer_prefix(clusters, d_model, dw, dwo)
            got.append(s.export_cluster(0)[:2])
    for name, step, a, b in (("K", 2.0 ** -10, got[0][0], got[1][0]), ("V", 2.0 ** -7, got[0][1], got[1][1])):
        differ = float((a != b).mean())
        print(f"{name}: {differ:.2e} of the elements differ", flush=True)
        assert (np.abs(a - b) <= step * np.abs(b) + 2.0 ** -16).all() and differ <= 0.02


@pytest.mark.parametrize("d_model,n,Hq,choice", [(64, 160, 32, 2), (64, 55, 16, 0), (192, 160, 32, 0), (320, 160, 32, 0)])
def test_large_qkv_product_with_few_odd_steps(d_model, n, Hq, choice):
    """One, three and five contraction steps (10 240 x 6144 and 3520 x 4096): the queries of the batch."""
    Hkv, S = 8, 64
    assert tiles_of([n * S], (Hq + 2 * Hkv) * 128, d_model, 2 * Hkv * 128, SLOTS)[0] == choice
    g = torch.Generator(device="cuda:0").manual_seed(d_model)
    x = torch.randn((n * S, d_model), generator=g, device="cuda:0", dtype=torch.bfloat16)
    w = torch.randn(((Hq + 2 * Hkv) * 128, d_model), generator=g, device="cuda:0", dtype=torch.bfloat16) * d_model ** -0.5
    q = torch.zeros((n * S, Hq * 128), device="cuda:0", dtype=torch.bfloat16)
    params = sgc.make_params(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, io_dtype="bf16", max_position=256)
    ctx = sgc.sgc_ctx_create(params)
    nbytes = sgc.sgc_cache_pool_bytes(params, 1)
    pool = torch.zeros(nbytes, dtype=torch.uint8, device="cuda:0")
    cache = sgc.sgc_cache_create(ctx, pool.data_ptr(), nbytes, 1)
    sgc.sgc_cache_alloc_cluster(ctx, cache, 0, 16)
    plan = sgc.sgc_assign_clusters(ctx, cache, np.zeros(n, np.int32), np.full(n, S, np.int32), 1)[3]
    sgc.sgc_project_qkv_suffix(ctx, cache, plan, 0, x.data_ptr(), w.data_ptr(), d_model, q.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    sgc.sgc_plan_destroy(plan)
    sgc.sgc_cache_destroy(cache)
    sgc.sgc_ctx_destroy(ctx)
    _close(f"queries, contraction {d_model}", q, x.float() @ w[:Hq * 128].float().T)
