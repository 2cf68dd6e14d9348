"""The rotation of Q in front of its rounding to E4M3 is one stated fp32 operation per feature,
lo' = fma(lo, cos, -(hi sin)) and hi' = fma(lo, sin, hi cos), whatever the compiler would contract: which
product is rounded first decides now and then which code a value next to a rounding boundary gets.

The codes are read off the normaliser.  Key 0 has one feature set, every other key is zero, and the scale
makes key 0 outweigh them by more than 2^18: their probabilities round to zero, the row sum is 2^8 and the
normaliser is S_0 c ln 2, S_0 the two-term value of the query's feature.  Q holds pairs, found by search,
for which the two contractions give values at least 2e-5 apart; fp32 rounding of scale, product and
logarithm is 1e-6 at most."""
import numpy as np
import pytest
import torch

import pv_workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu
pv = pytest.importorskip("paper_2605_04263_amd.binding")

f32, f64 = np.float32, np.float64
FIRST_ROW = 17                         # the rows before it see few keys and are evaluated in fp32


def fma(a, b, c):
    return (a.astype(f64) * b.astype(f64) + c.astype(f64)).astype(f32)   # a has 8 bits: the sum is exact in fp64


def two_terms(x, partner):
    """Value that two E4M3 terms hold of x, with the power of two that the larger of the pair asks for."""
    amax = np.maximum(np.abs(x), np.abs(partner))
    fac = np.exp2(7 - np.floor(np.log2(amax.astype(f64)))).astype(f32)
    def e4m3(v):
        return torch.from_numpy(v).to(torch.float8_e4m3fn).float().numpy()
    y = x * fac
    top = e4m3(y)
    return (top + e4m3((y - top) * f32(16)) / f32(16)) / fac


def rotated(lo, hi, c, s):
    return fma(lo, c, -(hi * s)), fma(lo, s, hi * c)


def other_contraction(lo, hi, c, s):
    return fma(hi, -s, lo * c), fma(hi, c, lo * s)


@pytest.mark.parametrize("group", [1, 4, 7, 8])                 # query tiles, and one wave per head
@pytest.mark.parametrize("half", [0, 1])
def test_codes_of_rotated_q(group, half):
    n, col = 500, 3
    pr = wl.Problem([60], [n - 60], [0], [1], [[]])
    w = wl.make_custom(pr, group, 1, 128, dtype=torch.bfloat16, rope_theta=5e5, seed=3)
    ver = gc.make_verifier(pv, w)
    ver.build_mask()
    dev = ver.device
    k = torch.zeros(n, 1, 128, dtype=torch.uint8)
    k[0, 0, col + 64 * half] = 0x38                              # 1.0
    k_scale = 64.0
    scales = torch.tensor([k_scale], dtype=torch.float32, device=dev)
    v = torch.full((n, 1, 128), 0x38, dtype=torch.uint8, device=dev)
    lse = torch.zeros(group, n, dtype=torch.float32, device=dev)

    def run(q):
        out = torch.zeros(n, group, 128, dtype=torch.float32, device=dev)
        pv.pv_masked_attention_fp8kv(ver.sizes, ver.plan, q.to(dev), k.to(dev), v, scales, scales, out, ver.workspace,
                                     lse, softmax_scale=1.0, rope_theta=w.rope_theta)
        torch.cuda.synchronize()

    run(w.q)                                                     # leaves the table of (cos, sin) in the workspace
    table = ver.workspace.view(torch.uint8)[:n * 64 * 8].view(torch.float32).reshape(n, 64, 2)[:, col].cpu().numpy()

    rng = np.random.default_rng(11 + half)
    rows, pairs, apart = [], [], []
    for _ in range(16):
        m = 1 << 20
        r = rng.integers(FIRST_ROW, n, size=m)
        lo, hi = (torch.from_numpy(rng.uniform(0.5, 2.0, size=m) * rng.choice([-1.0, 1.0], size=m)).to(torch.bfloat16)
                  .float().numpy() for _ in range(2))
        c, s = table[r, 0], table[r, 1]
        a, b = rotated(lo, hi, c, s), other_contraction(lo, hi, c, s)
        x, y = two_terms(a[half], a[1 - half]), two_terms(b[half], b[1 - half])
        ok = x > 0.5
        d = np.abs(x - y) > 2e-5 * np.abs(x)
        for i in np.nonzero(ok & d)[0]:
            rows.append(int(r[i])); pairs.append((lo[i], hi[i])); apart.append(True)
        for i in np.nonzero(ok)[0][:200]:
            rows.append(int(r[i])); pairs.append((lo[i], hi[i])); apart.append(False)
    assert sum(apart) >= 20, sum(apart)

    todo = sorted(range(len(rows)), key=lambda i: not apart[i])
    checked = 0
    while todo and checked < 2000:
        q, used, later = torch.zeros(n, group, 128, dtype=torch.bfloat16), {}, []
        for i in todo:
            head = next((h for h in range(group) if (rows[i], h) not in used), None)
            if head is None:
                later.append(i)
                continue
            used[rows[i], head] = i
            q[rows[i], head, col], q[rows[i], head, col + 64] = float(pairs[i][0]), float(pairs[i][1])
        run(q)
        got = lse.cpu().numpy()
        at = list(used)
        r = np.array([x[0] for x in at]); h = np.array([x[1] for x in at])
        p = np.array([pairs[used[x]] for x in at], dtype=f32)
        both = rotated(p[:, 0], p[:, 1], table[r, 0], table[r, 1])
        want = two_terms(both[half], both[1 - half]).astype(f64) * k_scale
        err = np.abs(got[h, r] - want) / want
        assert err.max() <= 5e-6, (err.max(), int((err > 5e-6).sum()), len(at))
        checked += len(at)
        todo = later
        if not any(apart[i] for i in todo):
            break
