"""The launch that appends and attends: no workgroup reads a row of the cache that the call appends without having appended it
itself (the kernel's own arithmetic, on the CPU)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fresh_plan") / "fresh_plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2507_11830_amd", "csrc"),
                    os.path.join(ROOT, "tests", "fresh_plan_host.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def shared_batch(rng):
    """Lengths and a block table in which prefixes lie on pages of their own, on other sequences' cached pages and on pages whose rows
    (some or all) the call appends."""
    batch = int(rng.integers(1, 7))
    ctx, new = np.zeros(batch, np.int32), rng.integers(0, 200, batch).astype(np.int32)
    pages = []
    free = list(rng.permutation(400))
    for s in range(batch):
        row = []
        if s and rng.random() < 0.8:  # the first tokens are another sequence's
            o = int(rng.integers(s))
            row = pages[o][: int(rng.integers(0, len(pages[o]) + 1))]
            # a page that both append to would get two contents: the prefix covers the shared pages whole
            ctx[s] = 16 * len(row) + int(rng.integers(0, 40))
        else:
            ctx[s] = int(rng.integers(0, 300)) if rng.random() < 0.6 else 0
        need = -(-int(ctx[s] + new[s]) // 16)
        pages.append(row + [free.pop() for _ in range(need - len(row))])
    table = np.full((batch, max(1, max(map(len, pages)))), -1, np.int32)
    for s, row in enumerate(pages):
        table[s, : len(row)] = row
    return ctx, new, table


def test_every_key_is_the_appended_one(plan):
    rng = np.random.default_rng(5)
    shared = 0
    for _ in range(400):
        ctx, new, table = shared_batch(rng)
        batch, max_pages = table.shape
        cu = np.concatenate([[0], np.cumsum(new)]).astype(np.int32) + int(rng.integers(0, 9))
        after = {}  # (page, row) -> new row, once the call is through
        for s in range(batch):
            for t in range(new[s]):
                p = int(ctx[s]) + t
                after[int(table[s, p // 16]), p % 16] = int(cu[s]) + t
        rows = np.zeros((4096, 3), np.int32)
        ptr = lambda x: x.ctypes.data_as(ctypes.c_void_p)
        for s in range(batch):
            if new[s] == 0:
                continue
            own = {}
            if ctx[s] > 0:
                n = plan.appended(batch, int(new.max()), ptr(cu), ptr(ctx), ptr(table), max_pages, 400, s, ptr(rows))
                own = {(int(a), int(b)): int(c) for a, b, c in rows[:n]}
            for where, row in own.items():
                assert after[where] == row  # others append the same bytes
            below = 16 * plan.pool_pages(int(ctx[s]))
            assert below % 128 == 0 and below >= ctx[s]
            for p in range(int(ctx[s] + new[s])):
                where = int(table[s, p // 16]), p % 16
                if p < below:
                    assert after.get(where) == own.get(where)
                    shared += p < ctx[s] and where in own
                else:  # read from the new rows
                    assert after[where] == int(cu[s]) + p - int(ctx[s])
    assert shared > 1000


def test_sequences_without_cached_tokens_read_nothing_from_the_pool(plan):
    assert plan.pool_pages(0) == 0
    assert [plan.pool_pages(c) for c in (1, 128, 129)] == [8, 8, 16]
    assert plan.pool_pages(-5) * 16 > 1 << 30  # bad lengths: never the caller's buffer


@pytest.mark.parametrize("p,n,q,m,want", [(1000, 24, 1024, 8, 1), (1000, 25, 1024, 8, 0), (1024, 8, 1000, 24, 1), (1024, 8, 1000, 25, 0),
                                          (1000, 8, 1000, 8, 0), (1000, 100, 1010, 5, 0), (1010, 5, 1000, 100, 0)])
def test_buffers_that_share_bytes(plan, p, n, q, m, want):
    arg = [ctypes.c_void_p(p), ctypes.c_long(n), ctypes.c_void_p(q), ctypes.c_long(m)]
    assert plan.apart(*arg) == want
