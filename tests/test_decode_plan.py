"""Whether a decode step of few rows is one launch, against times measured for both ways (MI355X, microseconds a step, 16 steps): none may be
more than 5 % slower than the other way, the spread of such measurements.  Host only: the rule is part of the library, the
times are data."""
import ctypes

import numpy as np
import pytest

from paper_2505_10951_amd import sgc


def decode_plan(hq, hkv, clusters, steps=16, kv="bf16"):
    """{one launch, key ranges, row tiles} of a batch; clusters: (queries, their question tokens, prompt tokens)."""
    params = sgc.make_params(n_q_heads=hq, n_kv_heads=hkv, head_dim=128, n_layers=1, io_dtype="bf16", kv_dtype=kv, rope_base=10000.0)
    ctx = sgc.sgc_ctx_create(params)
    pages = sum(-(-P // 16) for _, _, P in clusters)
    nbytes = sgc.sgc_cache_pool_bytes(params, max(pages, 1))
    cache = sgc.sgc_cache_create(ctx, 0x7F0000000000, nbytes, len(clusters))          # (never dereferenced here)
    for c, (_, _, P) in enumerate(clusters):
        sgc.sgc_cache_alloc_cluster(ctx, cache, c, P)
    labels = np.repeat(np.arange(len(clusters), dtype=np.int32), [n for n, _, _ in clusters])
    lens = np.repeat(np.array([s for _, s, _ in clusters], np.int32), [n for n, _, _ in clusters])
    plan = sgc.sgc_assign_clusters(ctx, cache, labels, lens, len(clusters))[3]
    sgc.sgc_plan_enable_decode(ctx, plan, steps)
    out = np.zeros(3, np.int32)
    sgc.lib().sgc_debug_decode_plan(plan, out.ctypes.data_as(ctypes.c_void_p))
    sgc.sgc_plan_destroy(plan)
    sgc.sgc_cache_destroy(cache)
    sgc.sgc_ctx_destroy(ctx)
    return [int(x) for x in out]


@pytest.mark.parametrize("hq,hkv,clusters,one,two", [
    # clusters of uneven sizes: the step waits for the largest
    (32, 32, [(4, 186, 604), (9, 179, 604), (14, 188, 604), (7, 187, 604), (31, 200, 604), (5, 202, 604)], 101.0, 71.0),
    (32, 32, [(5, 318, 105), (8, 272, 105), (4, 293, 105), (4, 306, 105), (12, 274, 105), (25, 279, 105)], 104.3, 61.4),
    (8, 8, [(n, 55, 228) for n in (2, 1, 3, 9, 2, 3, 2, 2, 2, 20, 4, 6)], 25.1, 21.1),
    (8, 8, [(30, 189, 162), (6, 184, 229), (4, 186, 173), (5, 193, 221), (4, 193, 220), (14, 183, 213), (9, 190, 177), (3, 191, 163)], 32.1, 27.2),
    (32, 32, [(15, 148, 245), (9, 96, 283), (32, 130, 293)], 45.5, 38.7),
    (32, 32, [(9, 15, 457), (31, 18, 351), (15, 20, 363)], 26.1, 26.2),
    (32, 32, [(1, 417, 337), (1, 389, 896), (1, 249, 699), (5, 349, 825), (2, 303, 1026), (1, 452, 964), (1, 235, 436), (1, 423, 384)], 37.7, 49.5),
    # many own keys
    (8, 8, [(13, 262, 973), (13, 261, 648), (13, 260, 976), (12, 256, 391), (12, 264, 373), (12, 259, 431)], 25.5, 34.3),
    (8, 8, [(28, 120, 4268)], 24.1, 31.9), (32, 32, [(20, 399, 1460), (10, 501, 1460)], 53.0, 60.3),
    (32, 32, [(12, 240, 500)], 21.8, 28.6), (32, 32, [(12, 240, 500)] * 4, 46.7, 51.3), (32, 32, [(12, 475, 500)] * 4, 89.2, 98.0),
    (32, 8, [(8, 475, 2500)] * 4, 35.4, 42.9), (32, 32, [(32, 305, 500)] * 8, 311.3, 288.7), (32, 32, [(32, 305, 60)] * 8, 298.3, 274.0),
    # past a round of the chip's compute units
    (32, 32, [(32, 133, 80)] * 9, 201.5, 160.6), (32, 32, [(16, 20, 15)] * 9, 39.0, 32.8), (32, 32, [(20, 437, 25)] * 9, 329.8, 271.2),
    (32, 32, [(2, 68, 93), (2, 54, 128), (2, 159, 120), (1, 34, 70), (1, 157, 102), (1, 17, 67), (1, 140, 114), (1, 60, 81), (1, 77, 142)], 17.7, 25.6),
    (32, 32, [(7, 20, 1400)] * 10, 65.9, 56.8), (32, 32, [(5, 14, 120)] * 16, 23.7, 29.9), (32, 32, [(13, 28, 100)] * 20, 54.1, 60.3), (32, 32, [(20, 26, 96)] * 24, 99.9, 108.9),
    (32, 32, [(17, 30, 2200)] * 32, 307.1, 284.1), (32, 32, [(5, 180, 4300)] * 12, 215.9, 194.6),
    # the ordinary ones
    (32, 8, [(5, 29, 3001)], 15.1, 19.4), (32, 8, [(8, 100, 500)] * 4, 17.4, 19.9),
])
def test_the_faster_way(hq, hkv, clusters, one, two):
    few = decode_plan(hq, hkv, clusters)[0]
    assert (one if few else two) <= 1.05 * min(one, two)


@pytest.mark.parametrize("hq,hkv,clusters,kv,few,ranges,row_tiles", [
    (8, 8, [(32, 20, 600)], "bf16", 1, 8, 8), (8, 8, [(33, 20, 600)], "bf16", 0, 3, 8),             # 32 rows of a cluster and KV head, 33
    (8, 8, [(8, 20, 600)], "fp8_e4m3", 0, 3, 8),                                                     # an fp8 cache
    (8, 8, [(4, 40, 64)] * 32, "bf16", 1, 1, 256), (8, 8, [(4, 40, 64)] * 33, "bf16", 1, 1, 264),     # 256 row tiles, more of them
    (8, 8, [(14, 1, 64)] * 33, "bf16", 1, 1, 264), (8, 8, [(15, 1, 64)] * 33, "bf16", 0, 1, 264),   # ... of 14 rows and of 15
    (8, 8, [(15, 40, 64)] * 64, "bf16", 1, 1, 512), (8, 8, [(15, 40, 1000)] * 64, "bf16", 0, 1, 512),  # ... full rounds; over longer prompts
    (8, 8, [(5, 40, 1920)] * 33, "bf16", 1, 1, 264), (8, 8, [(5, 40, 1921)] * 33, "bf16", 0, 1, 264), # ... over 30 steps and 31
    (8, 8, [(1, 1, 200)] * 33, "bf16", 1, 1, 264), (8, 8, [(1, 1, 120)] * 33, "bf16", 0, 1, 264),     # ... of 10 units and of six
    (8, 8, [(10, 40, 64)] * 64, "bf16", 1, 1, 512), (8, 8, [(3, 40, 64)] * 65, "bf16", 0, 1, 520),    # past two rounds, few units a tile ...
    (8, 8, [(8, 40, 64)] * 128, "bf16", 1, 1, 1024), (8, 8, [(8, 40, 64)] * 129, "bf16", 0, 1, 1032), # ... and at the most row tiles there are counters for
])
def test_limits(hq, hkv, clusters, kv, few, ranges, row_tiles):
    assert decode_plan(hq, hkv, clusters, kv=kv) == [few, ranges, row_tiles]
