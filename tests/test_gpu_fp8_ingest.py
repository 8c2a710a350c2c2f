"""The two passes of an fp8 cache's ingest at prompt lengths around its pieces (pages of 16 tokens, chunks of 8 pages, more
chunks than a wavefront has lanes, and past 2048 pages longer chunks instead of more): scales and codes equal to the
oracle's, wherever in the prompt the largest value sits."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session  # noqa: E402


@pytest.mark.parametrize("d,kernel", [(128, sgc.SGC_KERNEL_AUTO), (64, sgc.SGC_KERNEL_GENERIC)])
@pytest.mark.parametrize("P", [1, 16, 127, 128, 129, 1000, 8209, 32768, 32769, 65600])
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


@pytest.mark.parametrize("d", [128, 64])
def test_codes_of_values_that_are_not_finite(d):
    """A NaN of either sign is code 0x7F and moves no scale; a head with an infinity has an infinite scale, under which
    its finite elements are zeros (with their sign) and the infinities NaN."""
    P = 40
    w = workloads.custom("fp8_not_finite", n_q_heads=2, n_kv_heads=2, head_dim=d, rope_base=0.0, io_dtype="bf16", kv_dtype="fp8_e4m3",
                         prefix_len=[P], cluster_sizes=[1], suffix_range=(2, 2), seed=d)
    nan = np.float32("nan")
    for poison in ([(0, 7, 3, nan), (1, 39, d - 1, -nan)], [(0, 0, 0, np.inf)], [(1, 17, 5, -np.inf), (0, 3, 3, -nan)]):
        arrays = list(w.prefix_kv(0))
        for x in arrays:
            for h, t, c, value in poison:
                x[t, h, c] = value
        with Session(w, kernel=sgc.SGC_KERNEL_AUTO if d == 128 else sgc.SGC_KERNEL_GENERIC) as s:
            s.alloc_cluster(0)
            s.prefix_prefill(0, k=arrays[0], v=arrays[1])
            gk, gv, ks, vs = s.export_cluster(0)
        for got, scale, x in ((gk, ks, arrays[0]), (gv, vs, arrays[1])):
            for h in range(2):
                y = x[:, h]
                if np.isinf(y).any():
                    assert np.isinf(scale[h])
                    ref = np.where(np.signbit(y), 0x80, 0)
                else:
                    codes, ref_scale, _ = orc.quantise_e4m3(np.where(np.isnan(x), 0, x)[:, h:h + 1].astype(np.float64))
                    assert scale[h] == ref_scale.astype(np.float32)[0]
                    ref = codes[:, 0]
                assert np.array_equal(got[:, h], np.where(np.isfinite(y), ref, 0x7F)), (h, poison)
