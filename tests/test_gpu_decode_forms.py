"""GPU parity of the decode kernels' divisions of the keys — workgroups with equal shares of the batch's keys, splits
of a workgroup, splits of one wave — at the lengths and batch sizes where each can go wrong.  The tolerance is the
repository's (bf16 result and weights, fp32 sums)."""
import numpy as np
import pytest

from harness import TOL
from test_gpu_parity import custom_workload, run_chunk_steps, run_full_compare, run_fused_steps

pytestmark = pytest.mark.gpu

# around every page, block, four-block round and row-cost boundary; rows far longer than a workgroup's share; none
EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 0, 255, 256, 257, 383, 384, 385, 511, 512, 513, 640, 641, 3000, 5, 9001, 0]
BATCHES = {
    "edges": EDGES,
    "one": [2500],
    "one-block": [20],
    "slot-of-sequences": list(range(1, 65)),
    "two-slots": [0] * 63 + [700, 64, 1300] + [33] * 10,
    "most-sequences": [40 + 7 * (i % 13) for i in range(512)],
    "too-many-for-shares": [40 + 7 * (i % 13) for i in range(513)],
}


@pytest.fixture(params=[1, 2, 3], ids=["one-wave", "shares", "splits"])
def form(request):
    import paper_2507_11830_amd as sp

    sp.sp_debug_set_tuning("decode_form", request.param)
    yield request.param
    sp.sp_debug_set_tuning("decode_form", 0)


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (6, 2, 64), (32, 8, 128)])
@pytest.mark.parametrize("batch", sorted(BATCHES))
def test_decode_forms(form, batch, Hq, Hkv, d):
    lens = np.array(BATCHES[batch])
    lens = lens[: 70] if Hq == 32 else lens
    keep = lens > 0
    w = custom_workload(f"form{form}-{batch}-{Hq}-{Hkv}-{d}", lens, np.maximum(lens - 1, 0), Hq, Hkv, d, "prefill", seed=201)
    if keep.all():
        run_full_compare(custom_workload(w.name, lens, lens - 1, Hq, Hkv, d, "decode", seed=201), check_cache=False)
        run_fused_steps(custom_workload(w.name + "-fused", lens, lens - 1, Hq, Hkv, d, "decode", seed=202))
    else:
        decode_with_empty(w, lens)


def decode_with_empty(w, lens):
    """sp_attn_decode on a batch with sequences of length 0, whose output rows are zeros."""
    import torch

    import paper_2507_11830_amd as sp
    from harness import GpuRunner, OracleRunner, bits_of, dev_i32, report_err, to_dev
    from workloads import normal_bf16

    g, o = GpuRunner(w), OracleRunner(w)
    for st in w.steps():
        g.append(st)
        o.append(st)
    q = normal_bf16(np.random.default_rng(5), (len(lens), w.Hq, w.d))
    want = o.o.attn_decode(o.kp, o.vp, q, lens.astype(np.int32), w.block_table, w.scale)
    out = torch.full((len(lens), w.Hq, w.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((sp.sp_attn_decode_workspace_size(len(lens), int(lens.max()), w.Hq, w.d),), 0xFF, dtype=torch.uint8, device="cuda")
    sp.sp_attn_decode(g.cache, to_dev(q), out, dev_i32(lens), g.bt, int(lens.max()), float(w.scale), ws)
    torch.cuda.synchronize()
    assert report_err(w.name, bits_of(out), want) <= TOL
    assert not bits_of(out)[lens == 0].any()


# query tokens per sequence and cached tokens: chunks that straddle block, page and share boundaries, empty chunks
CHUNKS = {
    "ragged": ([4, 1, 0, 3, 4, 2, 4, 4, 0, 1], [0, 30, 64, 126, 127, 255, 1021, 4000, 12, 9000]),
    "all-empty-but-one": ([0, 0, 3, 0], [50, 60, 1500, 70]),
    "one-long": ([4], [12001]),
}


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (8, 2, 64), (32, 8, 128)])
@pytest.mark.parametrize("chunks", sorted(CHUNKS))
def test_short_chunk_forms(form, chunks, Hq, Hkv, d):
    """The same divisions with several query tokens per sequence, with one column tile and (4 heads per KV head, 16
    tokens) with two."""
    new, ctx = (np.array(x) for x in CHUNKS[chunks])
    run_chunk_steps(custom_workload(f"chunk{form}-{chunks}-{Hq}-{Hkv}-{d}", ctx + new, ctx, Hq, Hkv, d, "prefill", seed=203))
    if Hq // Hkv == 4:
        new = 4 * new - (new > 1)
        run_chunk_steps(custom_workload(f"chunk2-{form}-{chunks}-{Hq}-{Hkv}-{d}", ctx + new, ctx, Hq, Hkv, d, "prefill", seed=204))
