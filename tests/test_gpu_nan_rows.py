"""A NaN in one query row stays in that row: the row sums of two queries share a column of the matrix
product that forms them, and must not share its NaN.  (The kernels may re-centre the exponent of a row
whose neighbour is not finite, so the other rows agree to rounding, not to the bit: two roundings of P to
bf16 (2^-8 each) or to E4M3 (see test_gpu_attention_fp8: 8e-2 at most per run) apart.)"""
import pytest
import torch

import pv_workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (5, 1, 128), (8, 1, 128), (4, 1, 64)])
def test_nan_query_row(hq, hkv, d, fp8):
    if fp8 and d != 128:
        pytest.skip("the FP8 path is built for head size 128")
    pr = wl.Problem([40], [300], [2], [24], [[90, 300]])
    w = wl.make_custom(pr, hq, hkv, d, dtype=torch.bfloat16, rope_theta=5e5, seed=71)
    ver = gc.make_verifier(pv, w)
    ver.build_mask()
    dev = ver.device

    def run(q):
        out = torch.zeros(q.shape, dtype=torch.float32, device=dev)
        lse = torch.zeros(hq, pr.total_tokens, dtype=torch.float32, device=dev)
        if fp8:
            kc, ksc = wl.quantize_fp8(w.k)
            vc, vsc = wl.quantize_fp8(w.v)
            pv.pv_masked_attention_fp8kv(ver.sizes, ver.plan, q, kc.to(dev), vc.to(dev), ksc.to(dev), vsc.to(dev),
                                         out, ver.workspace, lse, rope_theta=w.rope_theta)
        else:
            ver.attention(q, w.k.to(dev), w.v.to(dev), out=out, lse=lse, rope_theta=w.rope_theta)
        torch.cuda.synchronize()
        return out, lse

    bad = [35, 100, 211, 339, 350]                   # rows of several tiles, either half of a tile
    q = w.q.to(dev)
    clean, clean_lse = run(q)
    q_nan = q.clone()
    q_nan[bad, :, 3] = float("nan")
    got, got_lse = run(q_nan)
    keep = torch.ones(pr.total_tokens, dtype=torch.bool, device=dev)
    keep[bad] = False
    assert torch.isnan(got[bad]).all() and torch.isnan(got_lse[:, bad]).all()
    assert torch.isfinite(got[keep]).all() and torch.isfinite(got_lse[:, keep]).all()
    tol = 1.6e-1 if fp8 else 2e-2
    assert (got[keep] - clean[keep]).abs().max() <= tol
    assert (got_lse[:, keep] - clean_lse[:, keep]).abs().max() <= tol
