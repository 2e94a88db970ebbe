"""GPU parity of sp_chunk_step where it appends inside the prefill launch (whole prompts of one length) and of the calls next to
that rule: outputs against the oracle, the cache image bit for bit, and the launches, read from a capture."""
import numpy as np
import pytest

from harness import TOL, GpuRunner, OracleRunner, bits_of, dev_i32, kernel_launches, report_err, to_dev
from test_gpu_parity import custom_workload

pytestmark = pytest.mark.gpu


def chunk_step(w, lo=0, hi=None, max_q=None, max_kv=None, launches=None):
    """The sequences lo..hi of w's last step by one sp_chunk_step, the rest of the batch by the oracle's own append."""
    import torch

    import paper_2507_11830_amd as sp

    hi = w.batch if hi is None else hi
    steps = list(w.steps())
    g, o = GpuRunner(w), OracleRunner(w)
    for st in steps[:-1]:
        g.append(st)
        o.append(st)
    st = steps[-1]
    o.append(st)
    want = o.attend(st)
    q = to_dev(st.q)
    k, v = (torch.cat([to_dev(x), torch.full((64, w.Hkv, w.d), float("nan"), dtype=torch.bfloat16, device="cuda")])[: q.shape[0]] for x in (st.k_new, st.v_new))
    out = torch.full_like(q, float("nan"))
    cu, ctx = dev_i32(st.cu_new)[lo : hi + 1], dev_i32(st.ctx_lens)[lo:hi]
    mq = max_q or int(st.new_lens[lo:hi].max())
    mkv = max_kv or int(st.seq_lens[lo:hi].max())
    sp.sp_debug_validate_hints(cu, ctx, q.shape[0], mq, mkv)
    need = sp.sp_attn_prefill_workspace_size(hi - lo, q.shape[0], mq, mkv, w.Hq, w.Hkv, w.d)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    call = lambda: sp.sp_chunk_step(g.cache, k, v, q, out, cu, ctx, g.bt[lo:hi], mq, mkv, float(w.scale), workspace=ws)
    call()
    torch.cuda.synchronize()
    a, b = int(st.cu_new[lo]), int(st.cu_new[hi])
    assert report_err(w.name, bits_of(out)[a:b], want[a:b]) <= TOL
    rest = torch.cat([out[:a], out[b:]])
    assert bool(rest.isnan().all())
    if (lo, hi) == (0, w.batch):
        gk, gv = g.cache_bits()
        assert np.array_equal(gk, o.kp) and np.array_equal(gv, o.vp), "cache image differs from the oracle's"
    else:
        gk, gv = g.cache_bits()
        for s in range(w.batch):
            for p in w.block_table[s, : -(-int(st.seq_lens[s]) // 16)] if lo <= s < hi else ():
                assert np.array_equal(gk[p], o.kp[p]) and np.array_equal(gv[p], o.vp[p])
    if launches is not None:
        assert [x for _, x in kernel_launches(call)] == launches


ONE, TWO = [(512, 1, 1)], [(256, 1, 1), (512, 1, 1)]


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (32, 8, 128), (2, 1, 64), (16, 2, 64), (64, 1, 64)])
@pytest.mark.parametrize("batch,n", [(1, 17), (1, 128), (3, 16), (2, 65), (1, 255), (3, 257), (1, 900)])
def test_whole_prompts_of_one_length(batch, n, Hq, Hkv, d):
    if n * (Hq // Hkv) <= 64:
        pytest.skip("served by the decode kernels")
    lens = np.full(batch, n)
    chunk_step(custom_workload(f"fresh-{batch}x{n}-{Hq}-{Hkv}-{d}", lens, 0 * lens, Hq, Hkv, d, "prefill", seed=n),
               launches=[(256, 1, 1)] if Hq == 64 and batch * n > 530 else ONE)  # more than a round of short halves: whole tiles


@pytest.mark.parametrize("Hq,Hkv,d,batch,n,threads", [(32, 8, 128, 3, 1057, 512), (16, 2, 64, 5, 1009, 256)])
def test_grids_that_fill_the_chip(Hq, Hkv, d, batch, n, threads):
    lens = np.full(batch, n)
    chunk_step(custom_workload(f"fresh-wide-{Hq}-{Hkv}-{d}", lens, 0 * lens, Hq, Hkv, d, "prefill", seed=5), launches=[(threads, 1, 1)])


@pytest.mark.parametrize("name,Hq,Hkv,d,new,ctx", [
    ("ragged", 8, 1, 128, [300, 299], [0, 0]),        # hints that leave room for a prefix
    ("prefix", 8, 1, 128, [300, 300], [0, 40]),
    ("no-groups", 4, 4, 128, [200, 200], [0, 0]),     # a query tile of 128 rows
    ("odd-groups", 6, 2, 64, [200, 200], [0, 0]),
])
def test_append_stays_a_launch_of_its_own(name, Hq, Hkv, d, new, ctx):
    new, ctx = np.array(new), np.array(ctx)
    chunk_step(custom_workload(f"not-fresh-{name}", new + ctx, ctx, Hq, Hkv, d, "prefill", seed=9), launches=TWO)


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (16, 2, 64)])
def test_sub_range_with_prefixes_under_large_hints(Hq, Hkv, d):
    """Hints that stand for more tokens than the range has do not rule out prefixes: the kernel meets some."""
    new, ctx = np.array([150, 64, 131, 55]), np.array([0, 100, 17, 0])
    w = custom_workload("fresh-sub", new + ctx, ctx, Hq, Hkv, d, "prefill", seed=31)
    chunk_step(w, lo=1, hi=3, max_q=200, max_kv=200, launches=ONE)
