"""The prefill form that cuts long work items, on the CPU: whatever the lengths are, its search deals out no more
workgroups than the host launches and no more partials than the workspace holds, and counts its pieces exactly."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2507_11830_amd as sp
from conftest import ROOT

SLOTS = 416
SHARDS = [(2, 1), (4, 1), (8, 1), (16, 2), (32, 8), (12, 3), (8, 8)]


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("cut_plan") / "cut_plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wno-unknown-pragmas",
                    "-I", os.path.join(ROOT, "paper_2507_11830_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cut_plan_host.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.launched_workgroups.argtypes = [ctypes.c_long] + [ctypes.c_int] * 4
    return L


@pytest.fixture(scope="module")
def plan(library):
    L = library

    def run(hq, hkv, ctx, new, slots=SLOTS):
        """(workgroups needed, launched, partials needed, partials counted, most pieces of an item)"""
        ctx, new = np.array(ctx, np.int32), np.array(new, np.int32)
        group = hq // hkv
        cols = group if group & (group - 1) == 0 else 1
        tpt, hgroups = 256 // cols, hq // cols
        launched = L.launched_workgroups(int(new.sum()), tpt, len(new), hgroups, slots)
        total = ctypes.c_int(-1)
        limit = L.limit_of(len(new), ctx.ctypes.data_as(ctypes.c_void_p), new.ctypes.data_as(ctypes.c_void_p),
                           tpt.bit_length() - 1, hgroups, slots, launched, ctypes.byref(total))
        pieces = []
        for c, n in zip(ctx.astype(np.int64), new.astype(np.int64)):
            keys = c + np.minimum(n, tpt * np.arange(1, -(-n // tpt) + 1))
            pieces.append(-(-(-(-keys // 64)) // limit))
        pieces = np.concatenate(pieces)
        return pieces.sum() * hgroups, launched, pieces[pieces > 1].sum() * hgroups, total.value * hgroups, pieces.max()

    return run


def check(got):
    needed, launched, partials, counted, most = got
    assert needed <= launched, f"{needed} workgroups dealt out, {launched} launched"
    assert partials == counted and partials <= SLOTS and most <= 16


@pytest.mark.parametrize("hq,hkv", SHARDS)
def test_batches_of_a_serving_engine(plan, hq, hkv):
    rng = np.random.default_rng(hq * 100 + hkv)
    for i in range(400):
        n = int(rng.integers(1, 257)) if i % 2 else int(rng.integers(1, 9))
        new = rng.integers(0, int(np.exp(rng.uniform(1, 8))) + 1, n)
        new[rng.integers(n)] += 1
        ctx = (np.exp(rng.uniform(0, np.log(1.3e5), n)) * (rng.random(n) < rng.choice([0.1, 0.9]))).astype(int)
        check(plan(hq, hkv, ctx, new))


# one sequence whose key tiles are more than the estimate can hold, alone and next to short ones
@pytest.mark.parametrize("hq,hkv", SHARDS)
@pytest.mark.parametrize("ctx", [1_300_000, 1_750_000, 3_500_000, 8_000_000, 16_700_000])
@pytest.mark.parametrize("new", [512, 4096, 10000])
def test_very_long_contexts(plan, hq, hkv, ctx, new):
    check(plan(hq, hkv, [ctx], [new]))
    check(plan(hq, hkv, [700, ctx, 0, 30000], [64, new, 900, 1]))


@pytest.mark.parametrize("batch,tokens,mq,mkv,heads", [(1, 64, 64, 5564, (8, 1, 128)), (2, 96, 60, 9000, (8, 1, 128)), (1, 512, 512, 33280, (16, 2, 64)), (4, 512, 128, 100128, (32, 8, 128))])
def test_slots_are_what_the_pieces_need(library, plan, batch, tokens, mq, mkv, heads):
    """No more slots than kMaxCutPieces of every item there may be, and enough for the search on any lengths of these hints."""
    slots = library.form_slots(batch, tokens, mq, mkv, *heads)
    items = tokens * heads[0] // 256 + batch * heads[1]
    assert 0 < slots <= min(SLOTS, 16 * items)
    assert slots <= library.merge_groups(batch, tokens, mkv, heads[0], heads[1])  # the merge covers every slot
    rng = np.random.default_rng(mkv)
    for _ in range(50):
        new = rng.multinomial(tokens - batch, [1 / batch] * batch) + 1 if batch > 1 else np.array([tokens])
        new = np.minimum(new, mq)
        ctx = rng.integers(0, mkv - new + 1)
        ctx[rng.integers(batch)] = mkv - mq
        unlimited, limited = plan(*heads[:2], ctx, new, SLOTS), plan(*heads[:2], ctx, new, slots)
        assert unlimited[2] == limited[2] <= slots and unlimited[0] == limited[0] <= limited[1]


def test_few_slots_and_wrong_hints(plan):
    """Fewer slots than pieces, or fewer workgroups than items: nothing is cut then rather than dropped."""
    for slots in (0, 1, 7, 60):
        needed, launched, partials, counted, _ = plan(8, 1, [9000, 100, 5000], [300, 40, 64], slots)
        assert partials == counted <= slots and needed <= launched


@pytest.mark.parametrize("hq,hkv,new,ctx", [(2, 1, 40000, 1_300_000), (8, 1, 10000, 1_750_000), (16, 2, 5000, 3_500_000)])
def test_such_contexts_keep_the_form_that_cuts_by_the_hints(hq, hkv, new, ctx):
    """... and the host does not ask for the cut form's workspace."""
    size = lambda: sp.sp_attn_prefill_workspace_size(1, new, new, ctx + new, hq, hkv, 128)
    auto = size()
    try:
        sp.sp_debug_set_tuning("prefill_cut", 1)
        assert auto == size()
    finally:
        sp.sp_debug_set_tuning("prefill_cut", 0)


S70, F8, W64 = (8, 1, 128), (32, 8, 128), (16, 2, 64)


@pytest.mark.parametrize("batch,tokens,mq,mkv,heads,cut", [
    # few query rows: pieces of 128 columns are shorter from about 12000 keys on
    (1, 64, 64, 5564, S70, True), (1, 64, 64, 4064, S70, False), (1, 64, 64, 20064, S70, False), (1, 64, 64, 131136, S70, False),
    (1, 256, 256, 5500, W64, True), (1, 256, 256, 100256, S70, False), (4, 236, 59, 41558, S70, False),
    # ... unless the merge of every row's pieces takes longer than that
    (7, 959, 137, 4660, (16, 2, 128), True),
    # ... and the same from about 24 query tiles on
    (1, 1024, 1024, 33024, S70, True), (4, 512, 128, 100128, F8, True),
    # chunks that leave most of a 256-column tile empty
    (64, 320, 5, 12005, W64, False), (64, 2368, 37, 6000, (12, 3, 64), False), (32, 1536, 48, 12048, (6, 2, 128), False),
    # many query tiles: what counts is the longest one against a CU's share
    (32, 13619, 512, 8704, S70, True), (33, 14100, 512, 8704, S70, True), (76, 9272, 122, 30976, (12, 3, 64), True),
    (24, 12288, 512, 4312, S70, False), (3, 3072, 1024, 4324, F8, False),  # of one length: up to 5 % slower cut
    (75, 4240, 110, 1700, S70, False), (134, 12000, 110, 1710, S70, False), (138, 40000, 400, 3200, S70, False),
    # without prefixes: one length, different lengths, on small grids and on full ones
    (1, 4097, 4097, 4097, W64, False), (1, 8183, 8183, 8183, S70, False), (2, 8200, 4887, 4887, S70, True),
    (1, 9560, 9560, 9560, S70, True), (4, 13124, 3281, 3281, S70, False), (2, 12704, 8250, 8250, S70, True),
])
def test_which_batches_take_the_form(library, batch, tokens, mq, mkv, heads, cut):
    assert (library.form_slots(batch, tokens, mq, mkv, *heads) > 0) == cut
