"""Host side of the prefill form that cuts long items: its tuning key and what it adds to the workspace size."""
import pytest

import paper_2507_11830_amd as sp


def test_tuning_key():
    L = sp.lib()
    for v, want in [(1, sp.SP_OK), (2, sp.SP_OK), (3, sp.SP_ERR_UNSUPPORTED), (-1, sp.SP_ERR_UNSUPPORTED), (0, sp.SP_OK)]:
        assert L.sp_debug_set_tuning(b"prefill_cut", v) == want


@pytest.mark.parametrize("batch,tokens,mq,mkv,heads,cut", [
    (32, 13000, 512, 8704, (8, 1, 128), True),     # few rounds of tiles on prefixes of any length
    (32, 13000, 512, 8704, (16, 2, 64), False),    # twice the tiles
    (32, 13000, 512, 2047, (8, 1, 128), False),    # short key ranges
    (257, 9000, 512, 8704, (8, 1, 128), False),    # more sequences than the search holds
    (4, 8192, 2048, 2048, (8, 1, 128), False),     # no prefix, short
    (2, 9000, 4887, 4887, (8, 1, 128), True),      # no prefix, long
    (64, 2111, 2048, 8000, (8, 1, 128), False),    # mixed
])
def test_workspace_has_room_for_the_partials(batch, tokens, mq, mkv, heads, cut):
    size = lambda: sp.sp_attn_prefill_workspace_size(batch, tokens, mq, mkv, *heads)
    auto = size()
    try:
        sp.sp_debug_set_tuning("prefill_cut", 1)
        never = size()
    finally:
        sp.sp_debug_set_tuning("prefill_cut", 0)
    room = 416 * (256 * (heads[2] + 2) * 4 + 32) + 256
    assert auto == (max(room, never) if cut else never)
