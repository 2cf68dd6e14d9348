"""Preparing a part of the tokens.  CPU (a host program over the library's own header): the launch is chosen by the keys
that it prepares, whatever the workspace holds, and its range has every key of the tokens and of the padding that goes
with them.  GPU: in workspaces of any capacity the blocks of the range hold what a preparation of everything writes and
every other byte is left alone."""
import os
import random
import subprocess

import pytest
import torch

import pv_workloads as wl
from paper_2605_04263_amd import build

pv = pytest.importorskip("paper_2605_04263_amd.binding")

PROGRAM = """
#include <cstdio>
#include "pv_internal.h"
int main() {
  long first, last, batch, keys;
  int hkv, d;
  while (std::scanf("%ld %ld %ld %ld %d %d", &first, &last, &batch, &keys, &hkv, &d) == 6) {
    const pv::PrepRange r = pv::prep_range(first, last, batch, keys);
    std::printf("%ld %ld %d\\n", (long)r.first, (long)r.last, pv::prep_heads(r.last - r.first, hkv, d));
  }
}
"""


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    at = tmp_path_factory.mktemp("range")
    (at / "range.hip").write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-host-only", "-x", "hip", "-std=c++17", "-I" + os.path.join(build.ROOT, "include"),
                    "-I" + build.CSRC, str(at / "range.hip"), "-o", str(at / "range")], check=True, capture_output=True)

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([str(at / "range")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


def test_heads_by_the_work(ranges):
    tokens = 3072
    for new, heads in ((512, 1), (3072, 1)):
        got = ranges([(tokens - new, tokens, 1, keys, 8, 128) for keys in (3072, 20480, 1 << 17)])
        assert {h for _, _, h in got} == {heads}
    # the end of a long request: as many heads as for a request of that length
    (_, _, part), (_, _, whole) = ranges([(60000, 65536, 1, 65536, 8, 128), (0, 5536, 1, 5568, 8, 128)])
    assert part == whole == 2


def test_range_has_every_key(ranges):
    rng = random.Random(3)
    rows, want = [], []
    for _ in range(400):
        lengths = [rng.choice([1, 15, 16, 17, 63, 64, 65, 100, 700]) for _ in range(rng.randint(1, 9))]
        start = [sum(lengths[:b]) for b in range(len(lengths) + 1)]
        pad = [sum((n + 63) // 64 * 64 for n in lengths[:b]) for b in range(len(lengths) + 1)]
        first, last = sorted(rng.randint(0, start[-1]) for _ in range(2))
        blocks = [pad[b] + i for b, n in enumerate(lengths) for i in range(0, pad[b + 1] - pad[b], 16)
                  if not (start[b] + min(i, n - 1) >= last or start[b] + min(i + 16, n) <= first)]
        rows.append((first, last, len(lengths), pad[-1], 8, 128))
        want.append((blocks, pad[-1]))
    for (first, last, _), (blocks, keys) in zip(ranges(rows), want):
        assert 0 <= first <= last <= keys and first % 16 == last % 16 == 0
        assert not blocks or first <= blocks[0] and blocks[-1] + 16 <= last


def up(n):
    return (n + 255) // 256 * 256


@pytest.mark.gpu
@pytest.mark.parametrize("hkv,d,lengths,first,last,extra", [
    (8, 128, [3000], 2500, 3000, 20480), (8, 128, [3000], 0, 3000, 64), (3, 64, [100, 64, 1, 700], 90, 170, 640),
    (8, 128, [33, 16, 900, 65], 49, 949, 128), (2, 128, [64, 64], 64, 64, 64), (1, 64, [129], 128, 129, 64),
    (8, 128, [6000], 1000, 6000, 9000 // 64 * 64), (16, 128, [300, 12000], 301, 302, 64), (8, 128, [24000], 100, 23999, 64)])
def test_part_of_the_tokens(hkv, d, lengths, first, last, extra):
    pr = wl.Problem([0] * len(lengths), lengths, [0] * len(lengths), [1] * len(lengths), [[]] * len(lengths))
    n, keys = pr.total_tokens, sum((x + 63) // 64 * 64 for x in lengths)
    capacity = keys + extra
    gen = torch.Generator(device="cuda").manual_seed(7)
    k, v = (torch.randn(n, hkv, d, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    ver = pv.Verifier(pr.prompt_len, pr.draft_len, pr.num_segments, pr.segment_len, pr.flat_boundaries(), hkv, hkv, d,
                      torch.bfloat16)
    ver.build_mask()
    size = pv.pv_prepared_workspace_bytes(ver.sizes, capacity)
    whole, part = (torch.full((size + 4096,), 0x7f, dtype=torch.uint8, device="cuda") for _ in range(2))
    pv.pv_prepare_kv(ver.sizes, ver.plan, k, v, whole[:size], 5e5, key_capacity=capacity)
    pv.pv_prepare_kv(ver.sizes, ver.plan, k, v, part[:size], 5e5, first_token=first, last_token=last, key_capacity=capacity)
    # blocks of 16 keys with a token of the range, or padding behind its last one
    inside = torch.zeros(capacity // 16, dtype=torch.bool)
    tokens = torch.zeros(capacity, dtype=torch.bool)
    pad = start = 0
    for x in lengths:
        for i in range(0, (x + 63) // 64 * 64, 16):
            if start + min(i, x - 1) < last and start + min(i + 16, x) > first:
                inside[(pad + i) // 16] = True
                tokens[start + min(i, x):start + min(i + 16, x)] = True
        pad += (x + 63) // 64 * 64
        start += x
    want = torch.full_like(whole, 0x7f)
    row = d * 4                                                      # bytes of a token's angles
    table = tokens.cuda()[:, None].expand(capacity, row).reshape(-1)
    want[:capacity * row][table] = whole[:capacity * row][table]
    at = up(capacity * row)
    block = hkv * capacity * d * 2
    # K: 16 bytes of each of 32 keys in turn; V^T: slabs of 16 keys
    in_keys = inside.cuda().view(1, capacity // 32, 1, 2, 1).expand(hkv, capacity // 32, d // 8, 2, 256).reshape(-1)
    in_slab = inside.cuda().view(1, capacity // 16, 1).expand(hkv, capacity // 16, 32 * d).reshape(-1)
    for mask in (in_keys, in_slab):
        want[at:at + block][mask] = whole[at:at + block][mask]
        at += up(block)
    assert torch.equal(part, want)
