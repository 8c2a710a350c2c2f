"""The two passes of an fp8 cache's ingest at prompt lengths around its pieces (pages of 16 tokens, chunks of 8 pages, more
chunks than a wavefront has lanes): scales and codes equal to the oracle's, wherever in the prompt the largest value sits."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session  # noqa: E402


@pytest.mark.parametrize("d,kernel", [(128, sgc.SGC_KERNEL_AUTO), (64, sgc.SGC_KERNEL_GENERIC)])
@pytest.mark.parametrize("P", [1, 16, 127, 128, 129, 1000, 8209])
def test_scales_and_codes_equal_the_oracle(P, d, kernel):
    Hkv = 2
    w = workloads.custom("fp8_ingest", n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=d, rope_base=0.0, io_dtype="bf16", kv_dtype="fp8_e4m3",
                         prefix_len=[P, 33], cluster_sizes=[1, 1], suffix_range=(2, 2), seed=P + d)
    with Session(w, kernel=kernel) as s:
        for c in range(2):
            s.alloc_cluster(c)
        for c in (1, 0):
            k, v = w.prefix_kv(c)
            n = k.shape[0]
            for h in range(Hkv):        # the largest magnitudes: first / last token, first / last channel, either sign
                k[(n - 1) * h, h, (d - 1) * (1 - h)] = -24.0 - h
                v[(n - 1) * (1 - h), h, (d - 1) * h] = 17.0 + h
            k[0, 0, 1] = -0.0
            s.prefix_prefill(c, k=k, v=v)
            gk, gv, ks, vs = s.export_cluster(c)
            for got, scale, x in ((gk, ks, k), (gv, vs, v)):
                codes, ref_scale, _ = orc.quantise_e4m3(x.astype(np.float64))
                assert np.array_equal(scale, ref_scale.astype(np.float32))
                assert np.array_equal(got, codes)
