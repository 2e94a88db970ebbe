"""GPU parity of sp_chunk_step where it appends inside the prefill launch (whole prompts of one length) and of the calls next to
that rule: outputs against the oracle, the cache image bit for bit, and the launches, read from a capture."""
import numpy as np
import pytest

from harness import TOL, GpuRunner, OracleRunner, bits_of, dev_i32, kernel_launches, report_err, to_dev
from test_gpu_parity import custom_workload

pytestmark = pytest.mark.gpu


def chunk_step(w, lo=0, hi=None, max_q=None, max_kv=None, launches=None, total=None, buffers=None):
    """The sequences lo..hi of w's last step by one sp_chunk_step, the rest of the batch by the oracle's own append.  total: tokens in
    the buffers, if more than the step has.  buffers: (k, v, out) -> the ones to use."""
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
    if total:
        q = torch.cat([q, torch.zeros((total - q.shape[0], w.Hq, w.d), dtype=q.dtype, device="cuda")])
    k, v = (torch.cat([to_dev(x), torch.full((64 + (total or 0), w.Hkv, w.d), float("nan"), dtype=torch.bfloat16, device="cuda")])[: q.shape[0]] for x in (st.k_new, st.v_new))
    out = torch.full_like(q, float("nan"))
    if buffers:
        k, v, out = buffers(k, v, out)
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


@pytest.mark.parametrize("Hq,Hkv,d,repeat,threads", [
    (8, 1, 128, 1, 512), (8, 2, 128, 1, 512), (8, 1, 64, 1, 512), (8, 2, 64, 1, 512),  # halved tiles
    (16, 2, 128, 1, 512), (8, 1, 128, 2, 512),  # whole tiles of 256 columns
    (16, 2, 64, 1, 256), (32, 2, 64, 1, 256),   # the four-wave kernel
])
@pytest.mark.parametrize("order", [1, -1])
def test_prefixes_that_the_call_appends(Hq, Hkv, d, repeat, threads, order):
    """Buffers and hints for more tokens than there are, and sequences whose cached tokens lie on pages that other sequences of the call
    append: those of a prompt, of a chunk on a prompt, and past a page of their own; with the streams' turn to the new rows in the
    first tiles, in the middle and behind the last one."""
    #      prompt, chunk on it, chunk on that one, own prefix, longer than the new rows, behind the last tile, a prompt
    new = np.array([333, 150, 61, 170, 9, 60, 350][::order] * repeat)
    ctx = np.array([0, 192, 320, 77, 300, 130, 0][::order] * repeat)
    w = custom_workload(f"fresh-shared-{Hq}-{Hkv}-{d}-{repeat}", new + ctx, ctx, Hq, Hkv, d, "prefill", seed=33)
    for r in range(repeat):
        a, b, c = (7 * r + (i if order == 1 else 6 - i) for i in range(3))
        w.block_table[b, : 192 // 16] = w.block_table[a, : 192 // 16]
        w.block_table[c, : 320 // 16] = w.block_table[b, : 320 // 16]
    chunk_step(w, max_q=400, max_kv=400, total=400 * len(new), launches=[(threads, 1, 1)])


@pytest.mark.parametrize("Hq,Hkv,d,threads", [(8, 1, 128, 512), (8, 2, 64, 512), (16, 2, 128, 512), (16, 2, 64, 256)])
def test_long_prefixes_that_the_call_appends(Hq, Hkv, d, threads):
    """The turn to the new rows in the middle of the tile loop."""
    new, ctx = np.array([700, 500, 300]), np.array([0, 640, 992])
    w = custom_workload(f"fresh-long-{Hq}-{Hkv}-{d}", new + ctx, ctx, Hq, Hkv, d, "prefill", seed=35)
    w.block_table[1, : 640 // 16] = w.block_table[0, : 640 // 16]
    w.block_table[2, : 992 // 16] = w.block_table[1, : 992 // 16]
    chunk_step(w, max_q=1300, max_kv=1300, total=3900, launches=[(threads, 1, 1)])


@pytest.mark.parametrize("Hq,Hkv,d,reuse", [(2, 2, 64, "k"), (2, 2, 64, "v"), (4, 1, 128, "v"), (4, 1, 128, None)])
def test_out_in_the_new_rows_buffers(Hq, Hkv, d, reuse):
    """The caller has no more use for the new rows once they are appended."""
    import torch

    def buffers(k, v, out):
        if reuse is None:
            return k, v, out
        big = torch.empty_like(out)  # the rows at its end
        rows = big.view(-1)[big.numel() - k.numel() :].view(k.shape)
        rows.copy_(k if reuse == "k" else v)
        return (rows, v, big) if reuse == "k" else (k, rows, big)

    lens = np.full(2, 300)
    chunk_step(custom_workload(f"fresh-reuse-{Hq}-{d}", lens, 0 * lens, Hq, Hkv, d, "prefill", seed=11), launches=TWO if reuse else ONE, buffers=buffers)


@pytest.mark.parametrize("which,launches", [("k", TWO), ("v", TWO), ("", ONE)])
def test_new_rows_off_a_16_byte_boundary(which, launches):
    import torch

    def moved(x):
        big = torch.empty(x.numel() + 4, dtype=x.dtype, device=x.device)
        big[4:] = x.reshape(-1)
        return big[4:].view(x.shape)

    lens = np.full(2, 300)
    chunk_step(custom_workload(f"fresh-moved-{which}", lens, 0 * lens, 8, 1, 128, "prefill", seed=13), launches=launches,
               buffers=lambda k, v, out: (moved(k) if which == "k" else k, moved(v) if which == "v" else v, out))


@pytest.mark.parametrize("Hq,Hkv,d,batch,n,threads", [
    (4, 4, 64, 2, 200, 512), (4, 4, 64, 1, 129, 512), (4, 4, 64, 12, 700, 256),  # 128 tokens a tile, 8 chunks each
    (4, 2, 128, 2, 200, 512), (4, 2, 128, 1, 65, 512),                           # 64 tokens, 16 chunks
])
def test_tiles_with_as_many_new_chunks_as_threads_move(Hq, Hkv, d, batch, n, threads):
    lens = np.full(batch, n)
    chunk_step(custom_workload(f"fresh-full-{Hq}-{Hkv}-{d}-{n}", lens, 0 * lens, Hq, Hkv, d, "prefill", seed=n), launches=[(threads, 1, 1)])


@pytest.mark.parametrize("Hq,Hkv,d,threads", [(2, 1, 128, 512), (2, 1, 64, 512), (8, 1, 128, 512), (16, 2, 64, 256)])
def test_prefixes_on_more_sequences_than_one_look_covers(Hq, Hkv, d, threads):
    """More (sequence, page) pairs than threads: every prompt has two chunks on it, one in front of it and one behind it in the batch."""
    new, ctx = np.array([40, 150, 90] * 14), np.array([96, 0, 112] * 14)
    w = custom_workload(f"fresh-many-{Hq}-{Hkv}-{d}", new + ctx, ctx, Hq, Hkv, d, "prefill", seed=37)
    for p in range(14):
        for reader, prompt in ((3 * p, 3 * (13 - p) + 1), (3 * p + 2, 3 * (13 - p) + 1)):
            w.block_table[reader, : ctx[reader] // 16] = w.block_table[prompt, : ctx[reader] // 16]
    chunk_step(w, max_q=210, max_kv=210, total=210 * len(new), launches=[(threads, 1, 1)])
