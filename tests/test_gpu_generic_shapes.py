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
