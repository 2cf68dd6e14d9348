"""A NaN in K or V reaches only the rows that share a key tile with it.

A row's probabilities at keys that it does not see are exactly zero, and a query tile (32 rows) reads only
the 64-key tiles that one of its rows sees: a NaN code beyond those must leave its rows as they are, also
where four query tiles of one head share a workgroup and with it the longer key list of their union.
Within a tile that a row does see, a NaN of V meets its zero probabilities: such rows are not checked."""
import numpy as np
import pytest
import torch

import pv_workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")

KEY_TILE, QUERY_TILE = 64, 32
NAN = 0x7F                                              # E4M3
# one request, and several whose last group of four query tiles is short
PROBLEMS = {
    "one": wl.Problem([40], [700], [3], [40], [[90, 300, 610]]),
    "three": wl.Problem([40, 3, 90], [300, 125, 410], [2, 0, 4], [24, 1, 33], [[90, 300], [], [50, 51, 200, 410]]),
}


def own_key_tiles(mask_of):
    """[row, key tile of the request], a request at a time: a row of the row's query tile sees a key of the tile."""
    tiles = []
    for m in mask_of:
        n = m.shape[0]
        per = [m[:, k:k + KEY_TILE].any(1) for k in range(0, n, KEY_TILE)]
        seen = np.stack(per, 1)
        for r in range(0, n, QUERY_TILE):
            seen[r:r + QUERY_TILE] = seen[r:r + QUERY_TILE].any(0)
        tiles.append(seen)
    return tiles


def masks(pr):
    flat, cut = gc.oracle_dense_mask_flat(pr), np.cumsum([pr.seq_len(b) ** 2 for b in range(pr.batch)])
    return [m.reshape(pr.seq_len(b), -1).astype(bool) for b, m in enumerate(np.split(flat, cut[:-1]))]


@pytest.mark.parametrize("where", ["k", "v"])
@pytest.mark.parametrize("name", list(PROBLEMS))
@pytest.mark.parametrize("group", [1, 2, 4, 5, 7, 8])
def test_fp8(group, name, where):
    pr, hkv = PROBLEMS[name], 2
    w = wl.make_custom(pr, group * hkv, hkv, 128, dtype=torch.bfloat16, rope_theta=5e5, seed=83)
    ver = gc.make_verifier(pv, w)
    ver.build_mask()
    dev = ver.device
    (kc, ksc), (vc, vsc) = wl.quantize_fp8(w.k), wl.quantize_fp8(w.v)

    def run(k, v):
        out = torch.zeros(w.q.shape, dtype=torch.float32, device=dev)
        lse = torch.zeros(w.q.shape[1], pr.total_tokens, dtype=torch.float32, device=dev)
        pv.pv_masked_attention_fp8kv(ver.sizes, ver.plan, w.q.to(dev), k.to(dev), v.to(dev), ksc.to(dev), vsc.to(dev),
                                     out, ver.workspace, lse, rope_theta=w.rope_theta)
        torch.cuda.synchronize()
        return out.cpu().numpy(), lse.cpu().numpy()

    clean, clean_lse = run(kc, vc)
    assert np.isfinite(clean).all()
    vis = masks(pr)
    own = own_key_tiles(vis)
    starts = np.cumsum([0] + [m.shape[0] for m in vis])
    for b, m in enumerate(vis):
        n = m.shape[0]
        for key in sorted({70, n // 2 + 5, n - 3, pr.prompt_len[b] + pr.draft_len[b] - 1}):
            codes = (kc if where == "k" else vc).clone()
            codes.view(torch.uint8)[starts[b] + key, :, 77] = NAN
            got, got_lse = run(codes, vc) if where == "k" else run(kc, codes)
            hit = np.zeros(pr.total_tokens, bool)
            hit[starts[b]:starts[b + 1]] = m[:, key]
            # K: every row that does not see the key; V: every row that does not share a key tile with it
            keep = np.ones(pr.total_tokens, bool)
            keep[starts[b]:starts[b + 1]] = ~m[:, key] if where == "k" else ~own[b][:, key // KEY_TILE]
            assert np.isnan(got[hit][..., 77 if where == "v" else slice(None)]).all(), (b, key)
            assert np.isfinite(got[keep]).all() and np.isfinite(got_lse[:, keep]).all(), (b, key)
            # V: the same operations, the same bits.  K: where a row of the tile does see the key, the tile's
            # probabilities are summed from their codes in fp32 instead of by the matrix instruction, which aligns
            # its addends to the largest and cuts what lies below: 2.4e-5 of the sum at most measured over these
            # cases, with the codes and the outputs' numerators the same.  The bound is ten times that.
            rel = 0.0 if where == "v" else 2.4e-4
            assert (np.abs(got[keep] - clean[keep]) <= rel * np.abs(clean[keep])).all(), (b, key)
            assert (np.abs(got_lse[:, keep] - clean_lse[:, keep]) <= rel).all(), (b, key)


# The bf16 kernels sum two queries of a tile in one column of a matrix product, so a NaN key that one of them sees
# reaches the other's sum and has to be taken out again; a row that does see it is NaN, in the whole pass and where the
# pieces of a segment row are merged.  |V| = 1: a row that is re-centred for its neighbour's sake rounds its
# probabilities to bf16 anew, 2^-8 of each at most, in either run.
@pytest.mark.parametrize("segments_only", [False, True])
@pytest.mark.parametrize("theta", [0.0, 5e5])
@pytest.mark.parametrize("group,d", [(1, 128), (4, 128), (5, 128), (8, 128), (4, 64), (5, 64)])
def test_bf16_keys(group, d, theta, segments_only):
    pr, hkv = PROBLEMS["three"], 2
    w = wl.make_custom(pr, group * hkv, hkv, d, dtype=torch.bfloat16, rope_theta=theta, seed=85)
    ver = gc.make_verifier(pv, w)
    ver.build_mask()
    dev = ver.device
    q, v = w.q.to(dev), torch.sign(w.v.float()).to(torch.bfloat16).to(dev)

    def run(k):
        out = torch.zeros(w.q.shape, dtype=torch.float32, device=dev)
        lse = torch.zeros(w.q.shape[1], pr.total_tokens, dtype=torch.float32, device=dev)
        (ver.segment_attention if segments_only else ver.attention)(q, k.to(dev), v, out=out, lse=lse, rope_theta=theta)
        torch.cuda.synchronize()
        return out.cpu().numpy(), lse.cpu().numpy()

    clean, clean_lse = run(w.k)
    assert np.isfinite(clean).all()
    vis = masks(pr)
    starts = np.cumsum([0] + [m.shape[0] for m in vis])
    delta = 2.0 ** -8
    for b, m in enumerate(vis):
        n, causal = m.shape[0], pr.prompt_len[b] + pr.draft_len[b]
        evaluated = np.zeros(pr.total_tokens, bool)
        for c in range(pr.batch):
            evaluated[starts[c] + (pr.prompt_len[c] + pr.draft_len[c] if segments_only else 0):starts[c + 1]] = True
        for key in sorted({20, 70, n // 2 + 5, causal - 1, causal, n - 3} & set(range(n))):
            bad = w.k.clone()
            bad[starts[b] + key, :, 33] = float("nan")
            got, got_lse = run(bad)
            hit = np.zeros(pr.total_tokens, bool)
            hit[starts[b]:starts[b + 1]] = m[:, key]
            hit &= evaluated
            keep = evaluated & ~hit
            assert np.isnan(got[hit]).all() and np.isnan(got_lse[:, hit]).all(), (b, key)
            assert np.isfinite(got[keep]).all() and np.isfinite(got_lse[:, keep]).all(), (b, key)
            assert np.abs(got[keep] - clean[keep]).max(initial=0) <= 2 * 2 * delta / (1 - delta) + 1e-5, (b, key)
            assert np.abs(got_lse[:, keep] - clean_lse[:, keep]).max(initial=0) <= -2 * np.log(1 - delta) + 1e-5, (b, key)
