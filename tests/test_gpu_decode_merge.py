"""GPU parity of the merge of decode partials where its forms change with the number of pieces: 16, 64 and 192 of them, and more than
one batch of loads."""
import numpy as np
import pytest

from test_gpu_parity import custom_workload, run_chunk_steps, run_full_compare

pytestmark = pytest.mark.gpu

# one sequence in pieces of 256 keys: 63, 64, 65, 96, 191 to 193 and 256 of them, the last one of a single key where it may be
ONE = [63 * 256, 64 * 256, 64 * 256 + 1, 96 * 256 - 1, 190 * 256 + 1, 192 * 256, 192 * 256 + 1, 256 * 256]


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (8, 1, 64)])
@pytest.mark.parametrize("lens", [[n] for n in ONE] + [[49000, 16, 5000], [70000] + [40] * 20])
def test_pieces_of_long_rows(lens, Hq, Hkv, d):
    lens = np.array(lens)
    run_full_compare(custom_workload(f"merge-{lens[0]}-{len(lens)}-{d}", lens, lens - 1, Hq, Hkv, d, "decode", seed=41), check_cache=False)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n", [64 * 256 + 1, 192 * 256 + 2])
def test_pieces_of_long_rows_under_several_tokens(n, d):
    lens, new = np.array([n, 700]), np.array([3, 1])
    run_chunk_steps(custom_workload(f"merge-tokens-{n}-{d}", lens, lens - new, 8, 1, d, "prefill", seed=42))
