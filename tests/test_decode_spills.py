"""The decode kernels' loops hold no spill code (a reload is paid for every block of keys), in the listings that the build
left behind."""
import glob
import os

import pytest

from paper_2507_11830_amd import build as b


@pytest.mark.parametrize("source,kernels", [("attn_decode", "decode_split_kernel"), ("attn_decode_stream", "decode_stream_kernel")])
def test_decode_loops_hold_no_spill_code(source, kernels):
    listings = glob.glob(os.path.join(os.path.dirname(b.__file__), "_build", source + "-hip-amdgcn-amd-amdhsa-gfx950.s"))
    if not listings:
        pytest.skip("no assembly listing from this build")
    counts = {k: n for k, n in b.loop_spills(listings[0]).items() if kernels in k}
    assert len(counts) >= 12
    for kern, n in counts.items():
        # the form at the register limit reloads per row segment, which is a loop around that over the blocks
        assert n <= (8 if "decode_stream_kernelILi128ELb1ELb1ELi2E" in kern else 0), (kern, n)
