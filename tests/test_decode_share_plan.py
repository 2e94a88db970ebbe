"""Equal shares of the decode, on the CPU: they hold all rows for every number of workgroups, also where the length hint
asked for fewer than the lengths need, and no row counts partials of workgroups that there are not."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from conftest import ROOT


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("share_plan") / "share_plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2507_11830_amd", "csrc"),
                    os.path.join(ROOT, "tests", "share_plan_host.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.share_of.argtypes = [ctypes.c_int, ctypes.c_long]
    L.one_wave.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long]
    return L


@pytest.mark.parametrize("wgs", [1, 2, 3, 5, 7, 64, 255, 256, 511, 512])
def test_shares_hold_all_rows(plan, wgs):
    rng = np.random.default_rng(wgs)
    totals = [1, 2, 19, 20, 21, 40, 41, 255, 256, 257, 5121, (1 << 26) + 1, (1 << 30) + 7]
    for total in totals + [int(x) for x in np.exp(rng.uniform(0, 20, 200))]:
        share = plan.share_of(total, wgs)
        assert share % 4 == 0 and share * wgs >= total, (total, wgs, share)


@pytest.mark.parametrize("wgs", [1, 2, 3, 256])
@pytest.mark.parametrize("lens", [[700], [64, 3000], [33] * 40 + [9000], [1] * 64])
def test_rows_count_partials_of_launched_workgroups_only(plan, wgs, lens):
    ends = np.cumsum([(n + 31) // 32 + 8 for n in lens])
    share = plan.share_of(int(ends[-1]), wgs)
    for end, n in zip(ends, lens):
        first_wg = (int(end) - (n + 31) // 32) // share  # of the row's first key block
        assert first_wg + plan.pieces_of(int(end), share, first_wg) <= wgs


@pytest.mark.parametrize("rows,geff,longest,d,splits,wave", [
    # many rows of a single short split, and of a few with one head per KV head
    (1024, 1, 128, 128, 1, True), (3752, 1, 121, 128, 1, True), (2048, 5, 66, 128, 1, True), (704, 4, 109, 128, 1, False),
    (2676, 1, 95, 64, 1, True), (1024, 8, 128, 64, 1, False), (1024, 1, 300, 128, 1, True), (1024, 4, 300, 128, 1, False),
    (1024, 1, 512, 128, 1, False), (128, 8, 100, 128, 1, False),
    # little data against shares and rounds that are not full
    (300, 8, 600, 128, 0, True), (200, 4, 1500, 64, 2, True), (256, 8, 900, 128, 1, False), (256, 4, 1500, 64, 2, False),
    (512, 8, 600, 128, 0, False), (384, 1, 900, 128, 0, True), (512, 2, 1849, 64, 0, True), (1024, 4, 1500, 128, 0, False),
    (16, 8, 8192, 128, 16, True), (64, 8, 8192, 128, 0, False), (2, 8, 16384, 128, 64, False),
])
def test_which_batches_stay_with_one_wave_splits(plan, rows, geff, longest, d, splits, wave):
    assert plan.one_wave(rows, geff, longest, d, splits) == wave
