"""Segment rows: the tiles that the segment-only call evaluates, the key pieces that the plan lists where the tiles are
few (they cover every tile's key list once, in pieces of nearly equal length, as many as there are places) and their
merged result against the oracle, at the group sizes of both numbers of places, with odd rows per piece, pieces of which
some rows see nothing, more tiles than a wave has lanes, lengths that take several rounds to find, and the list that a
launch of its own writes."""
import numpy as np
import pytest
import torch

import pv_workloads as wl
from tests.test_gpu_segment_attention import check_segments

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")


PROBLEMS = {
    "long_prompt": wl.Problem([3000], [40], [3], [17], [[0, 11, 40]]),
    "early_and_late": wl.Problem([5], [3000], [4], [17], [[1, 3, 2990, 3000]]),     # rows that see nothing of most pieces
    "no_prompt": wl.Problem([0], [2100], [3], [40], [[0, 1000, 2000]]),
    "two_requests": wl.Problem([700, 64], [1500, 3100], [3, 2], [32, 33], [[100, 101, 1500], [7, 3100]]),
    "segments_of_two_tiles": wl.Problem([101, 0], [400, 77], [5, 2], [64, 32], [[1, 300, 301, 399, 400], [30, 77]]),   # (too short to cut)
    "several_rounds": wl.Problem([1000], [12000], [6], [17], [[3, 2000, 2001, 6000, 9000, 12000]]),      # 200 lengths to try
    "two_rounds_exactly": wl.Problem([60000], [77], [2], [64], [[7, 77]]),
    "tiles_of_several_waves": wl.Problem([200, 9], [6000, 800], [100, 3], [32, 5], [[60 * (i + 1) for i in range(100)], [1, 9, 800]]),
    "launch_of_its_own": wl.Problem([100000, 3], [31300, 60], [5, 1], [9, 40], [[1, 9000, 9001, 31000, 31300], [60]]),
    "many_tiles": wl.Problem([130], [2500], [33], [32], [[75 * (i + 1) for i in range(33)]]),
}


def segment_tiles(pr):
    """{(request, first row of the listed tile): tile as the call evaluates it, or None}: the listed tiles with segment
    rows, cut at the segments' first rows where these are whole numbers of tiles long."""
    out, base = {}, pr.token_offsets()
    for b in range(pr.batch):
        p, t, s, n = pr.prompt_len[b], pr.draft_len[b], pr.segment_len[b], pr.seq_len(b)
        c = p + t
        for i, listed in enumerate(range(c // 32 * 32, n if pr.boundaries[b] else 0, 32)):
            t0 = c + 32 * i if s % 32 == 0 else listed
            rows = range(t0, min(t0 + 32, n))
            low = [r + 1 if r < c else p + pr.boundaries[b][(r - c) // s] for r in rows]
            own = [c + (r - c) // s * s for r in rows if r >= c]
            if not rows:
                out[b, listed] = None
                continue
            n_a = -(-max(low) // 64)
            jb0 = max(n_a, own[0] // 64)
            out[b, listed] = (base[b], t0, len(rows), min(low) // 64, n_a, jb0, max(jb0, rows[-1] // 64 + 1),
                              sum((pr.seq_len(x) + 63) // 64 * 64 for x in range(b)))
    return out


@pytest.mark.parametrize("name", list(PROBLEMS))
@pytest.mark.parametrize("hq,hkv", [(32, 8), (64, 8), (40, 8), (8, 8), (14, 2), (3, 3), (2, 1)])
def test_units(name, hq, hkv):
    pr = PROBLEMS[name]
    ver = pv.Verifier(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.flat_boundaries(), hq, hkv, 128,
                      torch.bfloat16)
    ver.plan.fill_(-1)
    ver.build_mask()
    blob = ver.plan.view(torch.int32).cpu().numpy()
    n, off, n_units, off_units, off_tiles = (int(blob[i]) for i in (30, 32, 36, 37, 38))
    assert n_units == ver.sizes.n_seg_pieces
    assert (ver.sizes.n_q_tiles > 4096) == (name == "launch_of_its_own")
    if name in ("several_rounds", "two_rounds_exactly", "launch_of_its_own") or name == "tiles_of_several_waves" and hkv in (1, 3):
        assert n_units > n
    want = segment_tiles(pr)
    assert len(want) == n
    if n_units == 0:                                             # uncut: found by the place of the listed tile
        for t in blob[off:off + 8 * n].reshape(n, 8).tolist():
            at = off_tiles + (t[7] + t[1]) // 32 * 8
            tile = want[pr.token_offsets().index(t[0]), t[1]]
            assert blob[at + 2] == 0 if tile is None else tuple(blob[at:at + 8].tolist()) == tile
        return
    units = blob[off_units:off_units + 12 * n_units].reshape(n_units, 12)
    seg = {t: 0 for t in want.values() if t is not None}
    used = units[units[:, 9] > 0]
    assert (units[:len(used), 9] > 0).all()
    lengths = {}
    for *tile, kt0, n_kt, piece, pieces in used.tolist():
        assert kt0 == seg[tuple(tile)] and 0 <= piece < pieces <= 8
        seg[tuple(tile)] += n_kt
        lengths.setdefault(tuple(tile), []).append(n_kt)
        assert piece == len(lengths[tuple(tile)]) - 1
    cost = {t: t[4] + t[6] - t[5] for t in seg}
    assert all(seg[t] == cost[t] and max(x) - min(x) <= 1 for t, x in lengths.items())
    length = min(x for x in range(min(4, max(cost.values())), max(cost.values()) + 1)
                 if sum(min(8, -(-c // x)) for c in cost.values()) <= n_units)
    assert all(len(lengths[t]) == min(8, -(-cost[t] // length)) for t in seg)


@pytest.mark.parametrize("hq,hkv,d,name", [(8, 2, 128, "long_prompt"), (8, 1, 128, "early_and_late"), (5, 1, 128, "no_prompt"),
                                           (2, 2, 64, "early_and_late"), (7, 1, 64, "two_requests"), (3, 1, 128, "two_requests"), (4, 1, 128, "segments_of_two_tiles"),
                                           (6, 1, 64, "segments_of_two_tiles")])
@pytest.mark.parametrize("theta", [0.0, 5e5])
def test_parity(hq, hkv, d, name, theta):
    pr = PROBLEMS[name]
    w = wl.make_custom(pr, hq, hkv, d, dtype=torch.bfloat16, seed=3, rope_theta=theta)
    ver = check_segments(w)
    assert (ver.sizes.n_seg_pieces > 0) == (name != "segments_of_two_tiles")


def test_parity_of_more_tiles_than_lanes():
    pr = wl.Problem([64], [3000], [80], [32], [[37 * (i + 1) for i in range(80)]])
    ver = check_segments(wl.make_custom(pr, 4, 1, 128, dtype=torch.bfloat16, seed=4, rope_theta=5e5), sample=160)
    assert 64 < ver.sizes.n_seg_tiles < ver.sizes.n_seg_pieces
