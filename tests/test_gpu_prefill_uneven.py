"""GPU parity of prefill batches without prefixes whose sequences differ in length and number a multiple of 8 streams, i.e. on
both sides of the rule that has their workgroups take items by rank (head groups, fill, shortest maximum)."""
import numpy as np
import pytest

from test_gpu_parity import custom_workload, run_full_compare

pytestmark = pytest.mark.gpu

LENS = {
    "uneven": [700, 3, 0, 129, 512, 64, 1, 300],
    "even": [600, 590, 600, 600, 580, 600, 599, 600],
    "short": [511, 3, 0, 129, 510, 64, 1, 300],
    "at-the-limit": [512] + [461] * 6 + [460],
}


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 1, 128), (4, 2, 64), (8, 8, 64)])
@pytest.mark.parametrize("lens", sorted(LENS))
def test_uneven_batches(lens, Hq, Hkv, d):
    n = np.array(LENS[lens])
    run_full_compare(custom_workload(f"uneven-{lens}-{Hq}-{Hkv}-{d}", n, 0 * n, Hq, Hkv, d, "prefill", seed=321))
