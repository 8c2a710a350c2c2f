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


def _close(name, got, ref):
    err = (got.float() - ref).abs()
    bar = 2.0 ** -8 * ref.abs() + 2.0 ** -15
    worst = float((err / bar).max())
    print(f"{name}: worst err/bar {worst:.3f}", flush=True)
    assert worst <= 1.0, name


# (rows, columns, heads of 128 = contraction / 128)
@pytest.mark.parametrize("M,N,Hq", [
    (1, 128, 1), (63, 128, 1), (64, 256, 3), (65, 384, 2),          # 64 x 64: two steps, fewer steps than stages, odd ones
    (129, 4096, 5), (300, 4096, 32),                                # 64 x 64 and 64 x 128
    (600, 4096, 32), (1000, 4096, 8),                               # 128 x 128, deep
    (2000, 4096, 32), (2048, 4096, 7),                              # 128 x 128, two workgroups per CU
    (4096, 4096, 32), (4300, 4096, 32), (5000, 4224, 16),           # 256 x 256 alone, and with a remainder
    (16384, 4096, 1), (16300, 4096, 2), (16384, 4096, 3),           # 256 x 256: fewer steps than the ring of slabs, and round it
])
def test_output_projection_rows_and_tiles(M, N, Hq):
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
    from test_gpu_layer import _run_layer
    prompt = workloads.custom("tiles", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16",
                              prefix_len=[rows, 0], cluster_sizes=[1, max(1, rows // 48)], suffix_range=(33, 64), seed=rows)
    last = prompt.n_queries - 1
    _run_layer(prompt, d_model, queries=sorted({0, last // 2, last}))


@pytest.mark.parametrize("d_model", [64, 192, 320])
def test_large_qkv_product_with_few_odd_steps(d_model):
    """One, three and five contraction steps in 256 x 256 tiles (10 240 rows, 6144 columns): the queries of the batch."""
    Hq, Hkv, n, S = 32, 8, 160, 64
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
