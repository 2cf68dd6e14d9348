"""CPU: the rule that cuts the segment-only call's tiles into key pieces looks at the requests that have such tiles.
Requests without a segment change nothing, a long one among them does not have short tiles cut, and a long judged
request keeps its pieces beside short ones, also where all tiles are more than the workgroups that run at once.
GPU: such batches against the oracle."""
import ctypes as C

import pytest
import torch

import pv_workloads as wl
from tests.test_gpu_segment_attention import check_segments

pv = pytest.importorskip("paper_2605_04263_amd.binding")

HEADS = [(32, 8), (64, 8), (40, 8), (8, 8), (16, 8), (14, 2), (3, 3)]


def batch(*requests):
    """(prompt, draft, segments, segment length) each, boundaries evenly spaced."""
    return wl.Problem([r[0] for r in requests], [r[1] for r in requests], [r[2] for r in requests],
                      [r[3] for r in requests], [[(j + 1) * r[1] // r[2] for j in range(r[2])] for r in requests])


def sizes(pr, hq, hkv):
    p = pv.make_problem(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.flat_boundaries())
    return pv.pv_query_sizes(p, hq, hkv, 128, pv.PV_BF16)


JUDGED = [(1000, 8000, 4, 32), (192, 8000, 10, 32), (500, 2500, 3, 17), (5, 2990, 4, 33), (300, 900, 2, 32)]


def test_sizes_keep_their_bytes():
    assert C.sizeof(pv.PvSizes) == 120


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("judged", JUDGED)
def test_requests_without_segments_change_nothing(judged, hq, hkv):
    alone = sizes(batch(judged), hq, hkv).n_seg_pieces
    for other in ((10, 40, 0, 1), (56, 200, 0, 1), (1000, 9000, 0, 1)):
        assert sizes(batch(judged, *[other] * 15), hq, hkv).n_seg_pieces == alone
        assert sizes(batch(*[other] * 3, judged, other), hq, hkv).n_seg_pieces == alone
    if judged == JUDGED[0] and hkv == 8:                  # 144 key tiles: always worth cutting
        assert alone > 0


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("short,n", [((40, 160, 2, 32), 15), ((40, 160, 3, 32), 10), ((30, 33, 1, 5), 3)])
def test_a_long_judged_request_beside_short_ones(short, n, hq, hkv):
    s = sizes(batch((1000, 8000, 3, 32), *[short] * n), hq, hkv)
    if s.n_seg_tiles * hkv < 512:                         # more places than tiles to give
        assert s.n_seg_pieces > s.n_seg_tiles
    else:
        assert s.n_seg_pieces == 0


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("s", [17, 32])
def test_keys_behind_the_boundaries_do_not_count(s, hq, hkv):
    early, late = (wl.Problem([24], [9000], [4], [s], [b]) for b in ([10, 20, 30, 40], [10, 20, 30, 9000]))
    assert sizes(early, hq, hkv).n_seg_pieces == 0        # two key tiles each
    assert sizes(late, hq, hkv).n_seg_pieces > 0


@pytest.mark.parametrize("change", [1, -1, 512])
def test_a_number_out_of_range_is_refused(change):
    s = sizes(batch(JUDGED[0]), 32, 8)
    s.n_seg_pieces = s.n_seg_tiles - 1 if change < 0 else pv.pv_query_sizes(
        pv.make_problem([1000], [8000], [4], [32], [2000, 4000, 6000, 8000]), 32, 8, 128, pv.PV_BF16).n_seg_tiles * 8 + change
    assert pv.lib.pv_static_workspace_needed(C.byref(s), C.byref(C.c_int64())) == pv.PV_ERR_SHAPE


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,pr", [
    (8, 2, batch(*[(10, 40, 0, 1)] * 2, (300, 2900, 3, 32), (56, 200, 0, 1))),
    (16, 2, batch((100, 3000, 2, 17), *[(20, 60, 3, 32)] * 46)),          # more tiles than a head's compute units
    (10, 2, batch(*[(20, 60, 2, 33)] * 44, (100, 3000, 2, 32))),
])
def test_parity(hq, hkv, pr):
    ver = check_segments(wl.make_custom(pr, hq, hkv, 128, dtype=torch.bfloat16, rope_theta=5e5, seed=5), sample=24)
    assert ver.sizes.n_seg_pieces > ver.sizes.n_seg_tiles
