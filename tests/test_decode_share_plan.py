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
