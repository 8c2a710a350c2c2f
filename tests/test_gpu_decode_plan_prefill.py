"""The suffix prefill of plans with decode steps: spare pages, kept for generated tokens, lie between the queries' own pages and
are none of its business, however many there are and whatever generated tokens have left in them."""
import numpy as np
import pytest

from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session, to_device, to_host_f32  # noqa: E402
from ref_util import oracle_suffix, tight_bar  # noqa: E402


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("cap", [20, 1000])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (2, 2)])
def test_generated_values_stay_out_of_a_second_prefill(hq, hkv, cap, kv):
    # several short queries to a tile, lengths around a page; what query 1 generates has infinite values
    lens = [3, 10, 16, 17, 1, 5, 15, 24]
    w = workloads.custom("spare", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", kv_dtype=kv, prefix_len=[40],
                         labels=np.zeros(len(lens), np.int32), suffix_len=np.array(lens, np.int32), seed=cap)
    _, ref, _ = oracle_suffix(w)
    bar = tight_bar(w, range(w.n_queries))[0] if kv == "bf16" else 6e-2
    with Session(w, kernel=sgc.SGC_KERNEL_MFMA) as s:
        s.alloc_cluster(0)
        s.prefix_prefill(0)
        s.assign()
        s.enable_decode(cap)
        dq, dk, dv = (to_device(x, "bf16") for x in w.suffix_qkv())
        first = to_host_f32(s.suffix_prefill(dq, dk, dv))
        assert np.abs(first - ref).max() <= bar
        for t in range(20):                      # past the page that the query's own tokens share with them
            q, k, v = (to_device(x, "bf16") for x in w.decode_qkv(t))
            v[1] = float("inf")
            s.decode_step(t, q, k, v)
        again = to_host_f32(s.suffix_prefill(dq, dk, dv))
        assert np.array_equal(first, again)
