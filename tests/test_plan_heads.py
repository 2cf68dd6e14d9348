"""A plan depends on the head counts only through the groups of four query tiles (n_quads): the segment-only call takes
plans that were built with the sizes of other head counts, whose list of key pieces has another number of places.
CPU: size and offsets.  GPU: such calls against the oracle, with guard bytes behind a workspace of the call's own size."""
import itertools

import pytest
import torch

import pv_workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_attention_bf16 import check_errors
from tests.test_gpu_segment_attention import segment_rows

pv = pytest.importorskip("paper_2605_04263_amd.binding")

PROBLEM = wl.Problem([512], [2048], [16], [32], [[128 * (i + 1) for i in range(16)]])       # 16 tiles, 48 key tiles
HEADS = [(32, 8), (8, 2), (16, 16), (32, 32), (40, 8), (8, 1)]


def sizes(pr, hq, hkv):
    prob = pv.make_problem(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.flat_boundaries(), pr.layout)
    return pv.pv_query_sizes(prob, hq, hkv, 128, pv.PV_BF16)


@pytest.mark.parametrize("pr", [PROBLEM, wl.Problem([3000], [40], [3], [17], [[0, 11, 40]]),
                                wl.Problem([300] * 40, [2200] * 40, [16] * 40, [32] * 40, [[2200] * 16] * 40)])
def test_plan_size_does_not_depend_on_the_heads(pr):
    by_quads = {}
    for hq, hkv in HEADS + [(16, 4), (4, 1), (1, 1), (24, 8), (64, 8), (28, 4), (1024, 1024)]:
        s = sizes(pr, hq, hkv)
        by_quads.setdefault(s.n_quads > 0, set()).add(s.plan_bytes)
    assert {k: len(v) for k, v in by_quads.items()} == {False: 1, True: 1}


@pytest.mark.parametrize("a,b", list(itertools.permutations([(32, 8), (8, 2), (4, 1), (64, 16), (16, 4)], 2)))
def test_sizes_with_other_heads_put_in(a, b):
    # one query for a model whose layers have different widths: the heads are replaced, the plan stays the same
    s, want = sizes(PROBLEM, *a), sizes(PROBLEM, *b)
    s.n_q_heads, s.n_kv_heads = b
    assert pv.pv_static_workspace_needed(s) == pv.pv_static_workspace_needed(want)
    capacity = s.padded_keys + 64
    assert pv.pv_prepared_workspace_bytes(s, capacity) >= pv.pv_prepared_workspace_bytes(want, capacity)
    room = pv.pv_prepared_workspace_bytes(s)
    assert room >= pv.pv_static_workspace_needed(s) + s.n_seg_pieces * b[0] * 32 * 130 * 4
    assert pv.pv_prepared_workspace_bytes(s, capacity) >= room


@pytest.mark.gpu
@pytest.mark.parametrize("put_in", [False, True])
@pytest.mark.parametrize("built,used", list(itertools.permutations(HEADS, 2)))
def test_segment_rows_under_a_plan_of_other_heads(built, used, put_in):
    w = wl.make_custom(PROBLEM, *used, 128, dtype=torch.bfloat16, rope_theta=5e5, seed=9)
    plan = pv.Verifier(PROBLEM.prompt_len, PROBLEM.draft_len, PROBLEM.num_segments, PROBLEM.segment_len,
                       PROBLEM.flat_boundaries(), *built, 128, torch.bfloat16)
    plan.plan.fill_(-1)
    plan.build_mask()
    s, dev = sizes(PROBLEM, *(built if put_in else used)), gc.device()
    s.n_q_heads, s.n_kv_heads = used
    room = pv.pv_prepared_workspace_bytes(s)
    ws = torch.full((room + 4096,), 0xA5, dtype=torch.uint8, device=dev)
    q, k, v = w.q.to(dev), w.k.to(dev), w.v.to(dev)
    out = torch.full(q.shape, 7.25, dtype=torch.float32, device=dev)
    pv.pv_segment_attention(s, plan.plan, q, k, v, out, ws[:room], rope_theta=5e5)
    torch.cuda.synchronize()
    assert bool((ws[room:] == 0xA5).all())
    rows = [segment_rows(PROBLEM)[0][::23]]
    check_errors(out[rows[0]].double().cpu().numpy(), gc.oracle_attention(w, rows_per_request=rows), bf16_out=False)
    assert bool((out[:PROBLEM.prompt_len[0] + PROBLEM.draft_len[0]] == 7.25).all())
    assert bool((out[PROBLEM.prompt_len[0] + PROBLEM.draft_len[0]:] != 7.25).any(-1).all())
