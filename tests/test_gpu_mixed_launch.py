"""GPU parity of mixed batches in the one-launch form (prefill and decode workgroups side by side): both widths of the prefill
workgroups, more decoding sequences than one per lane, rows in many shares, and a graph that replays it."""
import numpy as np
import pytest

from harness import TOL, GpuRunner, OracleRunner, bits_of, dev_i32, kernel_launches, report_err, to_dev
from test_gpu_parity import custom_workload, run_chunk_steps, run_full_compare

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(511)
# name: (Hq, Hkv, d, new tokens, cached tokens)
CASES = {
    "256-columns": (32, 8, 128, [1, 2400, 1, 3], [700, 0, 4000, 33]),
    "256-columns-d64": (32, 8, 64, [2400, 1, 1, 8], [100, 900, 3000, 1]),
    "many-decodes": (8, 1, 128, [1] * 130 + [300] + [1] * 20, list(RNG.integers(0, 900, 151))),
    "most-sequences": (8, 2, 64, [1] * 255 + [200], list(RNG.integers(0, 300, 256))),
    "long-rows": (8, 1, 128, [1, 90, 4], [20000, 77, 9000]),
    "no-keys-before": (8, 1, 64, [1, 0, 500, 1, 0, 2], [0, 40, 60, 0, 0, 0]),
    "odd-group": (6, 2, 128, [1, 200, 20, 1], [800, 100, 2000, 31]),  # the halves have 6 and 2 head groups; 20 tokens are too many for the decode half
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_mixed_launch(case):
    Hq, Hkv, d, new, ctx = CASES[case]
    new, ctx = np.array(new), np.array(ctx)
    w = custom_workload(f"mixed-launch-{case}", ctx + new, ctx, Hq, Hkv, d, "prefill", seed=311)
    run_full_compare(w, check_cache=False)
    run_chunk_steps(w)
    # one launch of both halves, then the merge over the decode half's rows
    found = launches(w, new, ctx)
    assert [block[0] for _, block in found][:1] == [512] and len(found) == 2, found
    assert found[1][0][:2] == (32 // min(Hq // Hkv, 32) * (Hq // Hkv), w.batch * Hkv), found


def launches(w, new, ctx):
    import torch

    import paper_2507_11830_amd as sp

    g = GpuRunner(w)
    for st in w.steps():
        g.append(st)
    q, cu, cx = to_dev(st.q), dev_i32(st.cu_new), dev_i32(st.ctx_lens)
    mq, mkv = int(new.max()), int((new + ctx).max())
    ws = torch.empty(sp.sp_attn_prefill_workspace_size(w.batch, q.shape[0], mq, mkv, w.Hq, w.Hkv, w.d), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)
    call = lambda: sp.sp_attn_prefill(g.cache, q, out, cu, cx, g.bt, mq, mkv, float(w.scale), workspace=ws)
    call()
    torch.cuda.synchronize()
    return kernel_launches(call)


def test_mixed_launch_in_a_graph():
    import torch

    import paper_2507_11830_amd as sp

    new, ctx = np.array([1, 1, 700, 1, 2]), np.array([700, 3000, 60, 15, 5000])
    w = custom_workload("mixed-graph", ctx + new, ctx, 8, 1, 128, "prefill", seed=312)
    g, o = GpuRunner(w), OracleRunner(w)
    for st in w.steps():
        g.append(st)
        o.append(st)
    want, q = o.attend(st), to_dev(st.q)
    cu, cx = dev_i32(st.cu_new), dev_i32(st.ctx_lens)
    ws = torch.empty(sp.sp_attn_prefill_workspace_size(5, q.shape[0], 700, 5002, 8, 1, 128), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)
    call = lambda: sp.sp_attn_prefill(g.cache, q, out, cu, cx, g.bt, 700, 5002, float(w.scale), workspace=ws)
    call()
    torch.cuda.synchronize()
    eager = bits_of(out).copy()
    assert report_err("mixed graph", eager, want) <= TOL
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            call()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        out.zero_()
        ws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits_of(out), eager), f"replay {rep} differs from the eager result"
