"""The order in which a launch takes its query tiles, at the edges of its three forms (one, two, three and
four workgroups for each of the 256 compute units): every row of every head against the fp64 oracle.  With
32 kv heads a compute unit's share is 8 tiles.  Tolerances: those of the bf16 and the FP8 path."""
import numpy as np
import pytest
import torch

import pv_workloads as wl
from oracle import pv_oracle as orc
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")

TILES = [8, 9, 16, 17, 20, 24, 25, 32, 33]


def problem(n_tiles):
    S = 20
    return wl.Problem([17], [32 * n_tiles - 17 - 3 * S - 5], [3], [S], [[9, 60, 100]])


@pytest.mark.parametrize("n_tiles", TILES)
def test_bf16(n_tiles):
    pr = problem(n_tiles)
    w = wl.make_custom(pr, 128, 32, 64, dtype=torch.bfloat16, rope_theta=5e5, seed=900 + n_tiles)
    ver = gc.make_verifier(pv, w)
    assert ver.sizes.n_q_tiles == n_tiles
    ver.build_mask()
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=ver.device)
    ver.attention(w.q.to(ver.device), w.k.to(ver.device), w.v.to(ver.device), out=out, rope_theta=w.rope_theta)
    torch.cuda.synchronize()
    err = np.abs(out.double().cpu().numpy() - gc.oracle_attention(w))
    assert err.max() <= 1e-2 and err.mean() <= 1e-3, (err.max(), err.mean())     # NaN fails both


@pytest.mark.parametrize("n_tiles", TILES)
def test_fp8(n_tiles):
    pr = problem(n_tiles)
    w = wl.make_custom(pr, 128, 32, 128, dtype=torch.bfloat16, rope_theta=5e5, seed=950 + n_tiles)
    kc, ksc = wl.quantize_fp8(w.k)
    vc, vsc = wl.quantize_fp8(w.v)
    ver = gc.make_verifier(pv, w)
    assert ver.sizes.n_q_tiles == n_tiles and ver.sizes.n_quads == 0     # one workgroup per tile and kv head
    ver.build_mask()
    dev = ver.device
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=dev)
    pv.pv_masked_attention_fp8kv(ver.sizes, ver.plan, w.q.to(dev), kc.to(dev), vc.to(dev), ksc.to(dev), vsc.to(dev),
                                 out, ver.workspace, None, rope_theta=w.rope_theta)
    torch.cuda.synchronize()
    ref = orc.masked_attention_fp8kv(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.boundaries,
                                     w.q.double().numpy(), kc.numpy(), vc.numpy(), ksc.numpy(), vsc.numpy(),
                                     rope_theta=w.rope_theta)
    err = np.abs(out.double().cpu().numpy() - ref)
    assert err.max() <= 8e-2 and err.mean() <= 5e-3, (err.max(), err.mean())
