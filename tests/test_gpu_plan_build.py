"""Plans at the edges of the ways to build them: the whole image or the request data alone in the kernel arguments of
the one launch, the request data uploaded before it, and, for more of them than a workgroup copies to LDS, separate
launches for the tiles and for their ranking; tile counts around a workgroup (256) and around what a ranking pass reads
(512), with a last wave of 1 to 4 tiles.  Each problem states the route that it is here for.  Everything is whole
numbers, against the oracle's mask and arrays."""
import numpy as np
import pytest
import torch

import pv_workloads as wl
from tests.test_gpu_mask_readout import check_plan, check_quad_list, check_work_list

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")

ARG_INTS, DATA_INTS, MAX_TILES = 896, 4096, 4096     # ints in kernel arguments; of request data, and tiles, in one launch


def even(lengths, k, s):
    """Requests of the given packed lengths with k segments of s tokens each."""
    return wl.Problem([9] * len(lengths), [n - 9 - k * s for n in lengths], [k] * len(lengths), [s] * len(lengths),
                      [[(j + 1) * (n - 9 - k * s) // (k + 1) for j in range(k)] for n in lengths])


WHOLE, IN_ARGS, UPLOADED, SEPARATE = "all in the arguments", "data in the arguments", "data uploaded before", "separate launches"
PROBLEMS = {
    "few_tokens_many_short_rows": (even([300] * 16, 2, 5), IN_ARGS),
    "few_tokens_data_too_large": (even([420] * 18, 40, 4), UPLOADED),
    "one_tile_requests": (even([32] * 70, 1, 3), UPLOADED),          # as many groups of tiles as tiles
    "one_tile_requests_in_arguments": (even([32] * 45, 1, 3), IN_ARGS),
    "tiles_256_one_workgroup": (even([192] * 16 + [160] * 32, 1, 7), IN_ARGS),
    "tiles_257_two_workgroups": (even([192] * 17 + [160] * 31, 1, 7), IN_ARGS),
    "tiles_256": (even([2720] * 3 + [32], 3, 7), WHOLE),
    "tiles_257": (even([2720] * 3 + [33], 3, 7), WHOLE),
    "tiles_512": (even([4096] * 4, 5, 33), WHOLE),
    "tiles_513": (even([4096] * 3 + [4097], 5, 33), WHOLE),
    "tiles_515_no_segments": (even([4096] * 4 + [70], 0, 1), WHOLE),
    "single_launch_256_tiles": (even([8187], 3, 64), WHOLE),         # tiles and groups of four side by side
    "single_launch_most_requests": (wl.Problem([0] * 50, [1] * 50, [0] * 50, [1] * 50, [[]] * 50), WHOLE),
    "separate_tiles_256": (even([2048] * 4, 1040, 1), SEPARATE),
    "separate_tiles_257": (even([2048] * 3 + [2049], 1040, 1), SEPARATE),
    "separate_tiles_512": (even([4096] * 4, 1040, 2), SEPARATE),
    "separate_tiles_513": (even([4096] * 3 + [4097], 1040, 2), SEPARATE),
    "separate_tiles_515": (even([4096] * 3 + [4192], 1040, 1), SEPARATE),
    "separate_two_tile_requests": (even([42] * 130, 30, 1), SEPARATE),
}


@pytest.mark.parametrize("name", list(PROBLEMS))
def test_plan(name):
    pr, route = PROBLEMS[name]
    ver = check_plan(pr)
    head = ver.plan.view(torch.int32)[:36].cpu().tolist()            # off_short at 18, off_device_begin at 19
    in_args, whole_image = head[18] <= ARG_INTS, head[19] <= ARG_INTS
    one_launch = ver.sizes.n_q_tiles <= MAX_TILES and head[18] <= DATA_INTS
    assert route == (SEPARATE if not one_launch else WHOLE if whole_image else IN_ARGS if in_args else UPLOADED), head[18:20]
    if "tiles_" in name and name.split("tiles_")[1].split("_")[0].isdigit():
        assert ver.sizes.n_q_tiles == int(name.split("tiles_")[1].split("_")[0])
    check_work_list(pr)
    check_quad_list(pr)


@pytest.mark.parametrize("name", list(PROBLEMS))
def test_segment_list(name):
    """The tiles that hold a segment row, longest first and otherwise in the order of the tile list."""
    pr, _ = PROBLEMS[name]
    ver = pv.Verifier(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.flat_boundaries(), 4, 2, 64,
                      torch.bfloat16)
    ver.plan.fill_(-1)
    ver.build_mask()
    blob = ver.plan.view(torch.int32).cpu().numpy()
    n_tiles, off_tiles, n_seg, off_seg = (int(blob[i]) for i in (4, 24, 30, 32))
    tiles = blob[off_tiles:off_tiles + 8 * n_tiles].reshape(n_tiles, 8)
    causal = dict(zip(np.cumsum([0] + [pr.seq_len(b) for b in range(pr.batch)]).tolist(),
                      [p + t for p, t in zip(pr.prompt_len, pr.draft_len)]))
    holds = np.array([t0 + rows > causal[base] for base, t0, rows in tiles[:, :3].tolist()])
    cost = tiles[:, 4] + tiles[:, 6] - tiles[:, 5]
    want = tiles[holds][np.argsort(-cost[holds], kind="stable")]
    assert n_seg == ver.sizes.n_seg_tiles == len(want)
    assert np.array_equal(blob[off_seg:off_seg + 8 * n_seg].reshape(n_seg, 8), want)
