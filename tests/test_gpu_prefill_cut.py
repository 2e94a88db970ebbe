"""GPU parity of the prefill form that cuts long work items by the lengths it finds on the device: every kind of
order (cut items of one and of several piece counts, uncut items behind them, several sequences per lane), the
tile counts on both sides of a cut, pieces that some rows see nothing of, head groups, and batches without any cut."""
import numpy as np
import pytest

from harness import TOL, GpuRunner, OracleRunner, bits_of, dev_i32, report_err, to_dev
from test_gpu_parity import custom_workload, run_chunk_steps, run_full_compare

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(411)
# name: (new tokens, cached tokens).  Ranges of up to 8 key tiles (512 keys) are never cut.
CASES = {
    "nothing-to-cut": ([300, 40, 0, 1], [200, 0, 30, 511]),
    "around-the-limit": ([1, 1, 1, 2, 33, 64, 65, 129], [511, 512, 513, 1023, 1000, 960, 960, 896]),
    "one-long": ([300], [5000]),
    "most-pieces": ([70], [11000]),
    "one-long-many-short": ([40] * 5 + [500] + [33] * 40, [100] * 5 + [3000] + [64] * 40),
    "no-prefix": ([1900, 700, 1, 0, 1300], [0, 0, 0, 0, 0]),
    "several-per-lane": (RNG.integers(0, 60, 150), RNG.integers(0, 1500, 150)),
}


@pytest.fixture(autouse=True)
def cut_everywhere():
    import paper_2507_11830_amd as sp

    sp.sp_debug_set_tuning("prefill_cut", 2)
    sp.sp_debug_set_tuning("prefill_short_chunk", 1)
    yield
    sp.sp_debug_set_tuning("prefill_cut", 0)
    sp.sp_debug_set_tuning("prefill_short_chunk", 0)


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (8, 2, 64), (6, 2, 128)])
@pytest.mark.parametrize("case", sorted(CASES))
def test_cut_items(case, Hq, Hkv, d):
    new, ctx = (np.array(x) for x in CASES[case])
    w = custom_workload(f"cut-{case}-{Hq}-{Hkv}-{d}", ctx + new, ctx, Hq, Hkv, d, "prefill", seed=301)
    run_full_compare(w)
    run_chunk_steps(w)


def test_cut_in_a_mixed_batch():
    import paper_2507_11830_amd as sp

    sp.sp_debug_set_tuning("prefill_short_chunk", 0)
    new, ctx = np.array([1, 1, 1, 900, 1, 4, 5]), np.array([700, 3000, 0, 2000, 15, 9000, 9])
    run_chunk_steps(custom_workload("cut-mixed", ctx + new, ctx, 8, 1, 128, "prefill", seed=302))


def test_cut_in_a_sub_range_and_in_a_graph():
    """Items are cut (the workspace says how many partials are in use), rows of other sequences stay untouched, and a
    captured launch replays bit for bit with stale workspace contents."""
    import torch

    import paper_2507_11830_amd as sp

    new, ctx = np.array([64, 200, 90, 30]), np.array([100, 4000, 2500, 50])
    w = custom_workload("cut-graph", ctx + new, ctx, 8, 1, 128, "prefill", seed=303)
    g, o = GpuRunner(w), OracleRunner(w)
    for st in w.steps():
        g.append(st)
        o.append(st)
    want, q = o.attend(st), to_dev(st.q)
    cu, cx, n = dev_i32(st.cu_new), dev_i32(st.ctx_lens), q.shape[0]
    mq, mkv = 200, 4200
    ws = torch.empty(sp.sp_attn_prefill_workspace_size(2, n, mq, mkv, 8, 1, 128), dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, -7.0)
    call = lambda: sp.sp_attn_prefill(g.cache, q, out, cu[1:4], cx[1:3], g.bt[1:3], mq, mkv, float(w.scale), workspace=ws)
    call()
    torch.cuda.synchronize()
    assert ws[:4].view(torch.int32).item() >= 2 * (200 + 90) // 32
    lo, hi = int(new[0]), int(new[:3].sum())
    eager = bits_of(out).copy()
    assert report_err("cut sub-range", eager[lo:hi], want[lo:hi]) <= TOL
    assert (out[:lo] == -7.0).all() and (out[hi:] == -7.0).all()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            call()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        out.fill_(-7.0)
        ws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits_of(out), eager), f"replay {rep} differs from the eager result"
