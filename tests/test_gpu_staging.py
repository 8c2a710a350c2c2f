"""The pinned buffers a call's tables are staged in are reused after eight copies, when the kernel that reads one has said so: with
the stream far behind the host, on one stream and on two in turn, every pass must still see its own tables."""
import numpy as np
import pytest

from paper_2505_10951_amd import sgc, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2505_10951_amd.harness import Session, to_device, to_host_f32  # noqa: E402


@pytest.mark.parametrize("n_streams", [1, 2])
@pytest.mark.parametrize("io,d", [("bf16", 128), ("f32", 64)])
def test_tables_of_queued_passes_stay_until_they_are_read(io, d, n_streams):
    w = workloads.custom("staging", n_q_heads=4, n_kv_heads=2, head_dim=d, rope_base=10000.0, io_dtype=io, prefix_len=[90, 33, 17],
                         cluster_sizes=[9, 5, 4], suffix_range=(1, 30), seed=3)
    rng = np.random.default_rng(1)
    cu, clusters = w.cu_seqlens, [0, 1, 2]
    q, k, v = w.suffix_qkv()
    batches = []
    for _ in range(14):                    # 28 copies and more through eight buffers, tables of very different sizes
        members = rng.permutation(w.n_queries)[: int(rng.integers(1, w.n_queries + 1))]
        rows = np.concatenate([np.arange(cu[n], cu[n + 1]) for n in members])
        batches.append((w.labels[members], w.suffix_len[members], [to_device(x[rows], io) for x in (q, k, v)]))
    pk = [[to_device(a, io) for a in w.prefix_kv(c)] for c in clusters]
    streams = [torch.cuda.Stream() for _ in range(n_streams)]

    def run(behind):
        # a session per stream: what a session stages on one stream is used on that stream
        sessions = [Session(w) for _ in streams]
        outs = []
        torch.cuda.synchronize()
        if behind:
            for st in streams:
                with torch.cuda.stream(st):
                    torch.cuda._sleep(100_000_000)
        for i, (labels, slen, (dq, dk, dv)) in enumerate(batches):
            s, st = sessions[i % n_streams], streams[i % n_streams]
            with torch.cuda.stream(st):
                for c in clusters:
                    s.alloc_cluster(c)
                sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, clusters, 0, None, [pk[c][0].data_ptr() for c in clusters],
                                               [pk[c][1].data_ptr() for c in clusters], None, None, s.stream)
                s.assign(labels, slen)
                outs.append(s.suffix_prefill(dq, dk, dv))
                for c in clusters:
                    s.free_cluster(c)
            if not behind:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        for s in sessions:
            s.close()
        return [to_host_f32(o) for o in outs]

    for a, b in zip(run(False), run(True)):
        assert np.isfinite(a).all() and np.array_equal(a, b)
