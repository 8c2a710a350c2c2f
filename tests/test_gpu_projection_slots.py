"""Where the projections' epilogues put keys and values: a batch's pages, whose questions begin and end at any row of a tile (pages that
lie inside a tile are written whole, others row by row, and the slots behind a question's last row are cleared), and prompts whose row
tiles travel with the launch (72 of them) or are copied to the device first (73)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_10951_amd import sgc, workloads
from paper_2505_10951_amd.harness import Session, to_device, to_host_f32
from test_gpu_layer import _check, _oracle_layer, _run_layer
from test_projection_plan import PAGES, SLOTS, plan as tiles_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d_model,T,choice", [
    (2, 1, 64, 300, 4), (4, 2, 4096, 1500, 3), (4, 2, 4096, 3500, 1), (16, 8, 64, 5000, 2), (16, 8, 64, 3500, 0),
])
def test_questions_at_any_row_over_pages_of_nan(Hq, Hkv, d_model, T, choice):
    """The pages held NaN in every slot before: what is not written or cleared shows."""
    n_kv = 2 * Hkv * 128
    assert tiles_of([T], Hq * 128 + n_kv, d_model, n_kv, SLOTS)[0] == choice
    rng = np.random.default_rng(T + choice)
    lens = []
    while sum(lens) < T:
        lens.append(int(min(T - sum(lens), rng.choice([1, 2, 15, 16, 17, 31, 32, 33, 48, rng.integers(1, 80)]))))
    w = workloads.custom("slots", n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=[0],
                         labels=[0] * len(lens), suffix_len=lens, seed=T)
    w_qkv, w_o = w.layer_weights(d_model)
    dwq, dwo = to_device(w_qkv, "bf16"), to_device(w_o, "bf16")
    # as many of the questions, spread over the batch, as there are near 200: with their neighbours they touch every kind of page
    queries = list(range(0, len(lens), max(1, len(lens) // 200)))
    _, ref = _oracle_layer(w, d_model, w_qkv, w_o, queries)
    with Session(w) as s:
        s.alloc_cluster(0)
        full = [(n + 15) // 16 * 16 for n in lens]
        s.assign(suffix_len=full)                # the same pages, every slot a row
        s.layer_suffix(torch.full((sum(full), d_model), float("nan"), dtype=torch.bfloat16, device="cuda:0"), d_model, dwq, dwo)
        torch.cuda.synchronize()
        s.assign()
        y = to_host_f32(s.layer_suffix(to_device(w.suffix_x(d_model), "bf16"), d_model, dwq, dwo))
        torch.cuda.synchronize()
    assert np.isfinite(y).all()
    for n in queries:
        _check(f"query {n}", y[int(w.cu_seqlens[n]):int(w.cu_seqlens[n + 1])], ref[n], abs_bar=2e-2, rel=2.0 ** -8)


@pytest.mark.parametrize("n", [72, 73])
def test_row_tiles_with_the_launch_and_copied(n):
    prompts = [5 + i % 7 for i in range(n)]
    assert tiles_of(prompts, 512, 64, 256, PAGES)[0] == 2        # one tile a prompt
    w = workloads.custom("row_tiles", n_q_heads=2, n_kv_heads=1, head_dim=128, rope_base=10000.0, io_dtype="bf16", prefix_len=prompts,
                         cluster_sizes=[1] * n, suffix_range=(3, 9), seed=n)
    with Session(w) as s:
        for c in range(n):
            s.alloc_cluster(c)
        dw, dwo = (to_device(x, "bf16") for x in w.layer_weights(64))
        s.layer_prefix(list(range(n)), 64, dw, dwo, with_output=False)
        assert sgc.lib().sgc_debug_carried(s.ctx) == (n <= 72)
    _run_layer(w, 64)
