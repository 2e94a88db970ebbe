"""GPU parity of the four-wave prefill kernel of head_dim 64 where its rounds of resident workgroups are dealt out: grids of just
over one round, within the second one, of counts that are no multiple of the XCDs, and beyond both."""
import numpy as np
import pytest

from test_gpu_parity import custom_workload, run_full_compare

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def whole_grids():
    import paper_2507_11830_amd as sp

    sp.sp_debug_set_tuning("prefill_split", 1)  # small grids would take the two-group kernel
    yield
    sp.sp_debug_set_tuning("prefill_split", 0)


@pytest.mark.parametrize("name,Hq,Hkv,new,ctx", [
    ("one-round", 16, 2, [640, 333, 17], [0, 0, 0]),            # 240 workgroups
    ("a-few-more", 16, 2, [700, 333, 17], [0, 0, 0]),           # 264
    ("second-round", 16, 2, [900, 333, 17], [0, 0, 0]),         # 342
    ("odd-counts", 5, 1, [700, 699, 1, 650, 33], [0] * 5),      # 25 streams, every head its own tiles
    ("both-rounds", 16, 2, [1100, 1090, 64, 700], [0] * 4),     # 552
    ("by-rank", 16, 2, [600, 310, 257, 31], [33, 500, 0, 1200]),
    ("xcd-streams", 12, 3, [300, 31, 290, 1, 64, 129, 33, 200], [0] * 8),  # 24 streams: three per XCD
])
def test_rounds_of_resident_workgroups(name, Hq, Hkv, new, ctx):
    new, ctx = np.array(new), np.array(ctx)
    run_full_compare(custom_workload(f"solo-{name}", new + ctx, ctx, Hq, Hkv, 64, "prefill", seed=77))


@pytest.mark.parametrize("new", [[700, 650], [330, 300, 340, 310]])  # with and without streams of their own for the XCDs
def test_chunk_hints_of_more_tiles_than_one_grid_dimension_holds(new):
    """32 heads a query tile leave it 4 tokens: 75000 tiles of a longest chunk of 300000, as a caller's fixed bound may be."""
    import torch

    import paper_2507_11830_amd as sp
    from harness import TOL, GpuRunner, OracleRunner, bits_of, dev_i32, report_err, to_dev

    new = np.array(new)
    w = custom_workload("solo-many-tiles", new, 0 * new, 64, 1, 64, "prefill", seed=79)
    g, o = GpuRunner(w), OracleRunner(w)
    (st,) = w.steps()
    o.append(st)
    q = to_dev(st.q)
    want = o.attend(st)
    for step in (False, True):  # attention after an append of its own, and with it
        out = torch.full_like(q, float("nan"))
        hint = 300000
        if step:
            sp.sp_chunk_step(g.cache, to_dev(st.k_new), to_dev(st.v_new), q, out, dev_i32(st.cu_new), dev_i32(st.ctx_lens), g.bt, hint, hint, float(w.scale))
        else:
            g.append(st)
            sp.sp_attn_prefill(g.cache, q, out, dev_i32(st.cu_new), dev_i32(st.ctx_lens), g.bt, hint, hint, float(w.scale))
        torch.cuda.synchronize()
        assert report_err(w.name, bits_of(out), want) <= TOL
