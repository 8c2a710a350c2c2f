"""Decode steps of few rows: a workgroup has one group of 32 rows and its eight wavefronts share the cached keys.  Sizes around a
wavefront's 32 keys, a page of 16 and the eight wavefronts' 256; up to 32 rows, and above that the 128-row workgroups; up to 128
tiles and above."""
import numpy as np
import pytest

pytest.importorskip("torch")

from paper_2505_10951_amd import workloads
from ref_util import oracle_caches
from test_gpu_decode import TOL, _oracle_decode, _run_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix", [[1, 15], [31, 33], [255, 256], [257, 300], [2000, 1]])
@pytest.mark.parametrize("hq,hkv,per", [(8, 2, 1), (8, 2, 8), (8, 2, 9), (8, 1, 4), (32, 32, 3), (160, 80, 16)])
def test_rows_and_keys_around_a_wavefront(hq, hkv, per, prefix):
    """(80 heads of two clusters: 160 tiles)"""
    w = workloads.custom("few", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=500000.0, io_dtype="bf16", prefix_len=prefix,
                         cluster_sizes=[per, per], suffix_range=(1, 20), seed=per, k_outlier_scale=8.0 if prefix[0] == 2000 else 1.0)
    o, lse = _run_decode(w, 2)[0]
    o_ref, lse_ref = _oracle_decode(w, 0, 2, oracle_caches(w, 0))
    assert np.isfinite(o).all() and np.abs(o - o_ref).max() <= TOL["bf16"] and np.abs(lse - lse_ref).max() <= 5e-2
