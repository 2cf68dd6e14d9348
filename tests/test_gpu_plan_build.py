"""Plans that are built by several launches, at the edges of their split: request data that fit the kernel
arguments of the launch that uses them or not, with and without rows behind them to upload; tile counts
around a workgroup (256), around what a ranking pass reads (512) and with a last wave of 1 to 4 tiles.
Everything is whole numbers, against the oracle's mask and arrays."""
import pytest

import pv_workloads as wl
from tests.test_gpu_mask_readout import check_plan, check_quad_list, check_work_list

pytestmark = pytest.mark.gpu


def even(lengths, k, s):
    """Requests of the given packed lengths with k segments of s tokens each."""
    return wl.Problem([9] * len(lengths), [n - 9 - k * s for n in lengths], [k] * len(lengths), [s] * len(lengths),
                      [[(j + 1) * (n - 9 - k * s) // (k + 1) for j in range(k)] for n in lengths])


PROBLEMS = {
    "few_tokens_many_short_rows": even([300] * 16, 2, 5),            # data in the arguments, short rows uploaded
    "few_tokens_data_too_large": even([420] * 18, 40, 4),            # request data beyond the arguments
    "one_tile_requests": even([32] * 70, 1, 3),                      # as many groups of tiles as tiles
    "tiles_256": even([2720] * 3 + [32], 3, 7),
    "tiles_257": even([2720] * 3 + [33], 3, 7),
    "tiles_512": even([4096] * 4, 5, 33),
    "tiles_513": even([4096] * 3 + [4097], 5, 33),
    "tiles_515_no_segments": even([4096] * 4 + [70], 0, 1),
    "single_launch_256_tiles": even([8187], 3, 64),                  # tiles and groups of four side by side
}


@pytest.mark.parametrize("name", list(PROBLEMS))
def test_plan(name):
    pr = PROBLEMS[name]
    check_plan(pr)
    check_work_list(pr)
    check_quad_list(pr)
