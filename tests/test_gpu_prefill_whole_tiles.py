"""GPU parity of small prefill grids on both sides of the rule that gives short key ranges whole query tiles instead of key tiles
halved over the wave groups, and the form each batch takes: its launches against those of either form by force."""
import numpy as np
import pytest

from harness import TOL, GpuRunner, OracleRunner, bits_of, dev_i32, kernel_launches, report_err, to_dev
from test_gpu_parity import custom_workload

pytestmark = pytest.mark.gpu

WHOLE, HALVES = 1, 2


@pytest.mark.parametrize("Hq,Hkv,d,new,ctx,form", [
    (8, 1, 128, [1024] * 4, [0] * 4, HALVES),                     # 256 workgroups: one round
    (8, 1, 128, [533] * 8, [0] * 8, WHOLE),                       # 266
    (8, 1, 128, [896] * 5, [0] * 5, WHOLE),                       # 280 and 14 key tiles
    (8, 1, 128, [897] * 5, [0] * 5, HALVES),                      # 15
    (32, 4, 128, [2170], [0], WHOLE),                             # 542: three rounds of halves
    (16, 2, 64, [129] * 18, [0] * 18, WHOLE),
    (16, 2, 64, [1150, 1140], [0, 0], HALVES),
    (16, 2, 128, [33, 400, 700, 577, 610], [0, 64, 1, 0, 17], WHOLE),
    (16, 2, 128, [256] * 10, [1300] * 10, HALVES),                # long prefixes
])
def test_form_and_parity(Hq, Hkv, d, new, ctx, form):
    import torch

    import paper_2507_11830_amd as sp

    new, ctx = np.array(new), np.array(ctx)
    w = custom_workload("whole-tiles", new + ctx, ctx, Hq, Hkv, d, "prefill", seed=3)
    g, o = GpuRunner(w), OracleRunner(w)
    for st in w.steps():
        g.append(st)
        o.append(st)
    want = o.attend(st)
    tol = max(TOL, np.abs(want).max() * 2.0**-8)  # rows of one or two keys reach 4, where half a bf16 unit is 2^-8 of the value
    q, cu, lens = to_dev(st.q), dev_i32(st.cu_new), dev_i32(st.ctx_lens)
    out = torch.empty_like(q)
    call = lambda: sp.sp_attn_prefill(g.cache, q, out, cu, lens, g.bt, int(new.max()), int((new + ctx).max()), float(w.scale))
    seen = {}
    for mode in (WHOLE, HALVES, 0):
        sp.sp_debug_set_tuning("prefill_split", mode)
        try:
            out.fill_(float("nan"))
            call()
            torch.cuda.synchronize()
            assert report_err(w.name, bits_of(out), want) <= tol
            seen[mode] = kernel_launches(call)
        finally:
            sp.sp_debug_set_tuning("prefill_split", 0)
    assert seen[WHOLE] != seen[HALVES] and seen[0] == seen[form]
