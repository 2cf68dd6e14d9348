"""Plans at the limits of the single launch: 4096 query tiles, 4096 ints of request data in LDS (896 of them in the
kernel arguments); and the list of rows with few keys, which the launch writes itself where every request starts with 16
such rows and has no others, and which is uploaded otherwise.  Whole numbers: the order of the tile lists follows from
the tile list, the rows from their definition."""
import numpy as np
import pytest
import torch

import pv_workloads as wl
from tests.test_gpu_mask_readout import check_work_order
from tests.test_gpu_plan_build import even

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")

PROBLEMS = {
    "tiles_4096": even([32768] * 4, 3, 40),
    "tiles_4097_separate_ranking": even([32768] * 3 + [32769], 3, 40),
    "one_request_beyond": even([131073 + 32], 7, 9),
    "data_4096_at_most": even([900] * 100, 25, 3),                      # uploaded, read from LDS
    "data_beyond_4096": even([900] * 100, 30, 3),
    "few_rows_of_some_requests": wl.Problem([0, 20, 3, 500] * 8, [9, 600, 700, 80] * 8, [2, 3, 4, 1] * 8, [7, 3, 30, 5] * 8,
                                            [[0, 5], [1, 2, 600], [0, 1, 20, 700], [80]] * 8),
    "sixteen_rows_each_on_average": wl.Problem([0, 1] * 20, [8, 400] * 20, [1, 0] * 20, [8, 1] * 20, [[8], []] * 20),
}


@pytest.mark.parametrize("name", list(PROBLEMS))
def test_lists(name):
    pr = PROBLEMS[name]
    ver = pv.Verifier(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.flat_boundaries(), 4, 2, 64,
                      torch.bfloat16)
    ver.plan.fill_(-1)
    ver.build_mask()
    blob = ver.plan.view(torch.int32).cpu().numpy()
    n, off_short, off_device, off_tiles, off_work, n_seg, off_seg = (int(blob[i]) for i in (4, 18, 19, 24, 25, 30, 32))
    if name.startswith("tiles_"):
        assert n == int(name.split("_")[1])
    if name.startswith("data_"):
        assert off_device > 896 and (off_short <= 4096) == (name == "data_4096_at_most")
    tiles, work = (blob[o:o + 8 * n].reshape(n, 8) for o in (off_tiles, off_work))
    check_work_order(tiles, work)
    base, rows, causal = pr.token_offsets(), [], {}
    for b in range(pr.batch):
        p, t, s = pr.prompt_len[b], pr.draft_len[b], pr.segment_len[b]
        causal[base[b]] = c = p + t
        rows += [(base[b] + i, base[b], 0, 0) for i in range(min(16, c))]
        rows += [(base[b] + c + k * s + a, base[b], p + x, c + k * s) for k, x in enumerate(pr.boundaries[b])
                 for a in range(s) if p + x + a + 1 <= 16]
    assert len(rows) == ver.sizes.n_short_rows
    assert np.array_equal(blob[off_short:off_short + 4 * len(rows)].reshape(-1, 4), np.array(rows))
    # tiles are listed request after request, 32 rows each, the last one of a request what is left
    want = [(base[b], t0, min(32, pr.seq_len(b) - t0)) for b in range(pr.batch) for t0 in range(0, pr.seq_len(b), 32)]
    assert np.array_equal(tiles[:, :3], np.array(want))
    holds = np.array([t0 + r > causal[x] for x, t0, r in want])
    cost = tiles[:, 4] + tiles[:, 6] - tiles[:, 5]
    assert n_seg == holds.sum()
    assert np.array_equal(blob[off_seg:off_seg + 8 * n_seg].reshape(n_seg, 8),
                          tiles[holds][np.argsort(-cost[holds], kind="stable")])
