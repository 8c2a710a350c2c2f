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


def test_waiting_for_a_stream_far_behind_does_not_wait_for_others():
    """The host waits for a staging buffer on a stream that is seconds behind; work of another stream that ends later is none of
    its business."""
    w = workloads.custom("behind", n_q_heads=4, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[40],
                         cluster_sizes=[1], suffix_range=(1, 2), seed=4)
    pk, pv = (to_device(a, "bf16") for a in w.prefix_kv(0))
    st, x = torch.cuda.Stream(), torch.zeros(64, device="cuda:0")

    def sleep(stream, cycles):
        with torch.cuda.stream(stream):
            torch.cuda._sleep(cycles)
            e = torch.cuda.Event(enable_timing=True)
            e.record()
        return e

    def independent(other):                    # (streams may share a hardware queue: work of one then waits for the other's)
        end = sleep(other, 100_000_000)
        with torch.cuda.stream(st):
            x.add_(1.0)
        st.synchronize()
        free = not end.query()
        torch.cuda.synchronize()
        return free

    with Session(w) as s:
        def one_copy():                        # page tables and jobs, each time
            s.alloc_cluster(0)
            sgc.sgc_prefix_prefill(s.ctx, s.cache, 0, 0, None, pk.data_ptr(), pv.data_ptr(), None, None, 40, st.cuda_stream)
            s.free_cluster(0)

        torch.cuda.synchronize()
        for _ in range(10):                    # all eight buffers are there
            one_copy()
        torch.cuda.synchronize()
        side = next((o for o in (torch.cuda.Stream() for _ in range(6)) if independent(o)), None)
        if side is None:
            pytest.skip("no stream that runs beside another")
        begin, end = sleep(st, 1), sleep(st, 100_000_000)
        torch.cuda.synchronize()
        cycles = 100_000_000 / begin.elapsed_time(end)          # a millisecond's
        mine, other = sleep(st, int(2500 * cycles)), sleep(side, int(4500 * cycles))
        for _ in range(9):                     # the ninth waits for the first, behind the sleep
            one_copy()
        assert mine.query() and not other.query()
        torch.cuda.synchronize()


@pytest.mark.parametrize("kv,n", [("bf16", 2), ("bf16", 14), ("fp8_e4m3", 2)])
def test_a_captured_call_is_replayed_and_its_buffer_used_again(kv, n):
    """Copies made while the stream is being captured say by an event that the buffer has been read (replays before it is used
    again see the call's own tables): the ingest that copies the tables itself, the general one, and the fp8 one."""
    w = workloads.custom("captured", n_q_heads=4, n_kv_heads=2, head_dim=128, rope_base=10000.0, io_dtype="bf16", kv_dtype=kv,
                         prefix_len=[90 - 5 * c for c in range(n)], cluster_sizes=[2] * n, suffix_range=(1, 30), seed=n)
    ids = list(range(n))
    pk, pv, pq = [[to_device(x, "bf16") for x in xs] for xs in ([w.prefix_kv(c)[0] for c in ids], [w.prefix_kv(c)[1] for c in ids], [w.prefix_q(c) for c in ids])]
    po = [torch.zeros_like(x) for x in pq]
    q, k, v = (to_device(x, "bf16") for x in w.suffix_qkv())
    o = torch.zeros_like(q)
    st = torch.cuda.Stream()
    ptr = lambda ts: [t.data_ptr() for t in ts]
    with Session(w) as s:
        def call():
            sgc.sgc_prefix_prefill_batched(s.ctx, s.cache, ids, 0, ptr(pq), ptr(pk), ptr(pv), ptr(po), None, st.cuda_stream)
            sgc.sgc_suffix_prefill_batched(s.ctx, s.cache, s.plan, 0, q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), None, st.cuda_stream)

        for c in ids:
            s.alloc_cluster(c)
        s.assign()
        torch.cuda.synchronize()
        for _ in range(2):                      # tables, blocks and buffers are there
            call()
        torch.cuda.synchronize()
        want = [to_host_f32(x) for x in po + [o]]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st, capture_error_mode="relaxed"):
            call()
        for _ in range(3):
            for x in po + [o]:
                x.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert all(np.array_equal(a, to_host_f32(b)) for a, b in zip(want, po + [o]))
        for _ in range(20):                     # every buffer again, the captured copy's among them
            call()
        torch.cuda.synchronize()
        assert all(np.array_equal(a, to_host_f32(b)) for a, b in zip(want, po + [o]))
