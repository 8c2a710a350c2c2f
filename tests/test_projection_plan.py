"""The tiles a projection is computed in, against times measured for every choice (MI355X, microseconds): no plan may be
slower than 256 x 256 tiles alone by more than 5 %, the spread of such measurements, nor than the best choice by more than 10 %.
Host only: the planner is part of the library, the times are data, those that its estimate was fitted to.  (The kernels have become
faster since, a batch's most; sgc_gemm.hip says beside the estimate where its choice is no longer the best one.)"""
import ctypes

import numpy as np
import pytest

from paper_2505_10951_amd import sgc

# choices: 0 = 256 x 256, 1 = 128 x 128 with a deep ring, 2 = 128 x 128 two to a CU, 3 = 64 x 128, 4 = 64 x 64;
# 10 + c = whole rounds of the chip in 256 x 256, the remaining rows in c
CHOICES = (0, 1, 2, 3, 4, 11, 12, 13, 14)
PLAIN, PAGES, SLOTS = 0, 0, 1           # where keys and values go (none, the cache's pages, the batch's slots)


def plan(prompts, N, K, n_kv, dest):
    """{first slabs in 256 x 256 tiles, kind of the rest} as one of CHOICES, and the number of slabs."""
    slabs = np.array([min(256, P - r) for P in prompts for r in range(0, P, 256)], np.int32)
    out = np.zeros(2, np.int32)
    p = ctypes.c_void_p
    sgc.lib().sgc_debug_projection_plan(slabs.ctypes.data_as(p), len(slabs), N, K, N - n_kv, dest, out.ctypes.data_as(p))
    big, rest = int(out[0]), int(out[1])
    return (0 if big == len(slabs) else rest if big == 0 else 10 + rest), len(slabs), big


@pytest.mark.parametrize("prompts,N,K,n_kv,dest,us", [
    ([16], 1024, 1024, 0, PLAIN, (21.6, 10.2, 9.7, 8.7, 6.5, 10.2, 9.7, 8.7, 6.9)),
    ([300], 4096, 4096, 0, PLAIN, (71.6, 33.5, 41.4, 21.2, 22.4, 33.1, 41.4, 21.2, 22.5)),
    ([1000], 4096, 4096, 0, PLAIN, (72.9, 40.4, 46.1, 45.4, 49.4, 38.7, 44.4, 45.3, 48.9)),
    ([2000], 4096, 4096, 0, PLAIN, (81.3, 77.9, 65.2, 89.6, 100.5, 79.5, 64.6, 88.5, 98.0)),
    ([8000], 640, 640, 0, PLAIN, (18.0, 15.9, 12.6, 22.1, 16.0, 15.7, 12.4, 22.1, 15.7)),
    ([5000], 4096, 4096, 0, PLAIN, (171.6, 192.6, 165.6, 226.7, 244.1, 146.3, 151.4, 150.3, 156.3)),
    ([12977], 4096, 4096, 0, PLAIN, (373.1, 504.4, 410.2, 561.4, 607.7, 350.5, 353.2, 351.4, 345.7)),
    ([16384], 4096, 4096, 0, PLAIN, (421.0, 619.5, 509.4, 698.6, 760.1, 416.5, 411.9, 411.9, 411.2)),
    ([300], 6144, 4096, 2048, PAGES, (95.7, 43.8, 50.9, 30.2, 31.0, 42.7, 50.9, 30.4, 31.2)),
    ([130] * 24, 6144, 1024, 2048, PAGES, (103.5, 108.2, 84.5, 129.8, 101.7, 117.0, 106.4, 110.6, 105.5)),
    ([2820], 6144, 4096, 2048, PAGES, (198.8, 192.0, 166.3, 204.9, 207.8, 159.8, 165.0, 144.7, 145.4)),
    ([1024] * 10, 10240, 1024, 2048, PAGES, (242.2, 296.3, 236.1, 473.8, 387.0, 254.5, 245.3, 260.6, 249.9)),
    ([130] * 24, 12288, 4096, 8192, PAGES, (491.3, 658.9, 527.1, 597.8, 618.5, 533.0, 510.0, 509.2, 498.2)),
    ([4000, 3999, 3601], 2048, 5120, 2048, PAGES, (248.0, 294.7, 246.0, 356.0, 375.4, 251.2, 230.9, 265.9, 270.3)),
    ([800], 12288, 1024, 8192, SLOTS, (56.3, 79.3, 64.4, 85.9, 58.1, 79.6, 64.5, 86.1, 58.2)),
    ([2400], 6144, 4096, 2048, SLOTS, (124.7, 166.8, 133.5, 188.9, 184.0, 168.2, 133.8, 189.6, 179.5)),
    ([6400], 6144, 1024, 2048, SLOTS, (122.9, 151.5, 118.3, 205.3, 153.6, 157.4, 141.3, 151.3, 139.8)),
    ([12800], 6144, 4096, 2048, SLOTS, (566.5, 765.7, 645.3, 873.7, 921.4, 608.2, 575.7, 605.8, 623.5)),
])
def test_plan_against_measured_times(prompts, N, K, n_kv, dest, us):
    choice, n_slabs, big = plan(prompts, N, K, n_kv, dest)
    assert 0 <= big <= n_slabs
    took = us[CHOICES.index(choice)]
    assert took <= 1.05 * us[0] and took <= 1.10 * min(us), choice
