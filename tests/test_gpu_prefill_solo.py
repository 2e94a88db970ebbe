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
