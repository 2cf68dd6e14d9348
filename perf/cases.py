"""Performance cases of the verification pass: what users of the library have it do, over its range.

A case names one call sequence on one packed batch:

  pass      one packed verification pass of a layer: mask plan, attention over every row, readout
            (segments = 0: the full-answer verification, a plain causal pass with no segment)
  segments  a judge pass whose prompt and draft rows exist already: mask plan, attention of the
            segment rows only, readout
  judge     the periodic judge pass of a serving engine: the keys of the prompt and of the draft's first
            part were prepared by an earlier pass and K/V live in a paged cache; mask plan, preparation of
            the new tokens' keys, segment rows, judge logits from the hidden states, decision

The lengths of a batch come from the case alone (`shape_seed` where they vary); the tensors from the
seed.  Everything is resident on the GPU before a pass, as it is between the layers of a model.
"""
from __future__ import annotations

import math
import random

import torch

import pv_workloads as wl
from paper_2605_04263_amd import binding as pv

PAGE = 64                    # tokens per page of the paged cache
HIDDEN = 4096                # hidden size in front of the judge's two lm-head rows
TAU = 0.985                  # judge confidence threshold of the readout


def _case(kind, batch, prompt, draft, segments, segment_len, heads, *, boundaries="uniform", theta=5e5,
          layout=0, fp8=False, outliers=False, lse=False, shape_seed=0, name=None):
    """prompt / draft / segments: one length for every request, or the (low, high) it is drawn from."""
    def ends(x):
        return (x, x) if isinstance(x, int) else x
    c = {"kind": kind, "batch": batch, "segment_len": segment_len, "boundaries": boundaries, "theta": theta,
         "q_heads": heads[0], "kv_heads": heads[1], "head_dim": heads[2], "layout": layout, "fp8": fp8,
         "outliers": outliers, "lse": lse, "shape_seed": shape_seed}
    for key, x in (("prompt", prompt), ("draft", draft), ("segments", segments)):
        c[key + "_min"], c[key + "_max"] = ends(x)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a short question with a short answer: four launches, latency is everything
        _case("pass", 1, 32, 256, 4, 16, (32, 8, 128), name="small_answer"),
        # the headline shape: one answer of 2048 tokens judged at 16 sentence-like boundaries
        _case("pass", 1, 512, 2048, 16, 32, (32, 8, 128), boundaries="sentences", shape_seed=2, name="answer_8b"),
        # the same packing with every segment behind the chunk it judges
        _case("pass", 1, 512, 2048, 16, 32, (32, 8, 128), boundaries="sentences", layout=1, shape_seed=2,
              name="answer_8b_interleaved"),
        # the full-answer judgment that precedes the packed pass
        _case("pass", 1, 512, 2048, 0, 1, (32, 8, 128), name="full_verify_8b"),
        # a serving batch: 16 requests of very different lengths
        _case("pass", 16, (128, 1024), (512, 4096), (4, 32), 32, (32, 8, 128), shape_seed=3, name="ragged_batch"),
        # group of five heads, outlier channels in K, no rotation
        _case("pass", 1, 1024, 4096, 32, 48, (40, 8, 128), boundaries="chunks", theta=0.0, outliers=True,
              shape_seed=4, name="answer_14b"),
        # long drafts of a large model, batch of 4: the largest
        _case("pass", 4, 2048, 8192, 64, 64, (64, 8, 128), shape_seed=5, name="long_batch_70b"),
        # K and V stored as FP8, the headline shape and the largest
        _case("pass", 1, 512, 2048, 16, 32, (32, 8, 128), boundaries="sentences", fp8=True, shape_seed=2,
              name="answer_8b_fp8"),
        _case("pass", 4, 2048, 8192, 64, 64, (64, 8, 128), fp8=True, shape_seed=5, name="long_batch_70b_fp8"),
        # premature verification while the draft grows, over a paged cache
        _case("judge", 1, 512, 2048, 16, 32, (32, 8, 128), boundaries="sentences", shape_seed=2, name="judge_8b"),
        # segment rows only for a serving batch (the full verification has been done)
        _case("segments", 16, (128, 1024), (512, 4096), (4, 32), 32, (32, 8, 128), shape_seed=3, name="segments_ragged"),
        # small heads, odd sizes, normalisers asked for
        _case("pass", 2, (211, 301), (1117, 1501), (7, 11), 23, (32, 8, 64), lse=True, shape_seed=6, name="small_heads"),
    ]


HEADS = [(32, 8), (32, 8), (40, 8), (64, 8), (64, 8), (8, 8), (16, 8), (24, 8), (48, 8), (28, 4)]


def draw(rng):
    """One more case of the same ranges: any call, group size, head size, packing and batch, lengths from
    a few dozen tokens to those of the largest listed case."""
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    limit = work(listed()[6])["flops"]
    while True:
        kind = rng.choice(["pass", "pass", "pass", "pass", "segments", "judge"])
        fp8 = kind == "pass" and rng.random() < 0.3
        hq, hkv = rng.choice(HEADS)
        d = 64 if not fp8 and rng.random() < 0.2 else 128
        batch = 1 if kind == "judge" else rng.choice([1, 1, 1, 2, 3, 5, 8, 16, 24])
        p, t = log_uniform(24, 2600), log_uniform(80, 9000)
        k = 0 if kind == "pass" and rng.random() < 0.15 else log_uniform(3, 64)
        if k > t // 4:
            continue
        s = rng.choice([16, 17, 24, 32, 33, 48, 64])
        ragged = batch > 1 and rng.random() < 0.7
        c = _case(kind, batch, (max(1, p // 3), p) if ragged else p, (max(4 * k, t // 4, 16), t) if ragged else t,
                  (k // 3, k) if ragged and kind == "pass" else k, s, (hq, hkv, d),
                  boundaries=rng.choice(["uniform", "sentences", "chunks"]), theta=rng.choice([0.0, 1e4, 5e5, 5e5]),
                  layout=1 if rng.random() < 0.2 else 0, fp8=fp8, outliers=rng.random() < 0.15,
                  lse=rng.random() < 0.25, shape_seed=rng.randrange(1 << 20))
        if c["draft_min"] <= c["draft_max"] and work(c)["flops"] <= limit:
            return c


def _problem(case):
    """Lengths and boundaries of every request, from the case alone."""
    r = random.Random(case["shape_seed"])
    ps, ts, ks, bounds = [], [], [], []
    for _ in range(case["batch"]):
        p = r.randint(case["prompt_min"], case["prompt_max"])
        t = r.randint(case["draft_min"], case["draft_max"])
        k = r.randint(case["segments_min"], case["segments_max"])
        if case["boundaries"] == "uniform":              # distinct positions anywhere in the draft
            b = sorted(r.sample(range(min(16, t - k), t + 1), k))
        elif case["boundaries"] == "sentences":          # gaps of sentence length
            b, x = [], 0
            for _ in range(k):
                x += max(1, int(r.gauss(0.75 * t / k, 0.1 * t / k)))
                b.append(min(t, x))
        else:                                            # equal chunks with jitter
            step = t / max(k, 1)
            b = sorted(max(1, min(t, int(step * (i + 1) + r.uniform(-step / 4, step / 4)))) for i in range(k))
        ps.append(p); ts.append(t); ks.append(k); bounds.append(b)
    return wl.Problem(ps, ts, ks, [case["segment_len"]] * case["batch"], bounds, case["layout"])


def _first_new_token(case, problem):
    """judge: the draft tokens before this one had their keys prepared by the previous judge pass."""
    return problem.prompt_len[0] + (3 * problem.draft_len[0]) // 4


def prepare(case, seed):
    problem = _problem(case)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    n, hq, hkv, d = problem.total_tokens, case["q_heads"], case["kv_heads"], case["head_dim"]

    def normal(*shape, dtype=torch.bfloat16):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dtype)

    st = {"case": case, "q": normal(n, hq, d), "k": normal(n, hkv, d), "v": normal(n, hkv, d)}
    if case["outliers"]:                                 # a few heavy-tailed channels per kv head
        channels = torch.randperm(d, generator=gen, device=dev)[:4]
        t3 = normal(n, hkv, 4, dtype=torch.float32) / normal(3, n, hkv, 4, dtype=torch.float32).square().mean(0).sqrt()
        st["k"][:, :, channels] = (4.0 * t3).to(torch.bfloat16)
    if case["fp8"]:
        st["k"], st["k_scale"] = wl.quantize_fp8(st["k"])
        st["v"], st["v_scale"] = wl.quantize_fp8(st["v"])
    ver = pv.Verifier(problem.prompt_len, problem.draft_len, problem.num_segments, problem.segment_len,
                      problem.flat_boundaries(), hq, hkv, d, torch.bfloat16, layout=case["layout"])
    st["ver"] = ver
    st["out"] = torch.zeros(n, hq, d, dtype=torch.bfloat16, device=dev)
    st["lse"] = torch.zeros(hq, n, dtype=torch.float32, device=dev) if case["lse"] else None
    st["logits"] = 4.0 * normal(problem.total_segments, 2, dtype=torch.float32)
    st["margin"] = pv.margin_from_tau(TAU)
    if case["kind"] == "judge":
        pages = (n + PAGE - 1) // PAGE
        table = torch.randperm(pages + pages // 4, generator=gen, device=dev)[:pages]
        for key in ("k", "v"):                           # the packed rows, scattered over the page pool
            rows = torch.zeros(pages * PAGE, hkv, d, dtype=torch.bfloat16, device=dev)
            rows[:n] = st[key]
            pool = torch.zeros(pages + pages // 4, PAGE, hkv, d, dtype=torch.bfloat16, device=dev)
            pool[table] = rows.view(pages, PAGE, hkv, d)
            st[key] = pool
        st["table"] = table.to(torch.int32)
        st["new"] = _first_new_token(case, problem)
        st["hidden"] = normal(n, HIDDEN)
        st["w2"] = normal(2, HIDDEN) * (1.0 / math.sqrt(HIDDEN))
        m = pv.margin_from_tau
        st["policy"] = pv.make_policy(m(TAU), m(0.9), m(0.998), m(0.97), [m(0.9)], 0.3, 3, 0.0, 3, premature=True)
        ver.build_mask()                                 # the previous pass: prompt and first part of the draft
        pv.pv_prepare_kv(ver.sizes, ver.plan, st["k"], st["v"], ver.workspace, case["theta"], 0, st["new"],
                         st["table"], PAGE)
    return st


def run(st):
    case, ver, theta = st["case"], st["ver"], st["case"]["theta"]
    ver.build_mask()
    if case["kind"] == "judge":
        pv.pv_prepare_kv(ver.sizes, ver.plan, st["k"], st["v"], ver.workspace, theta, st["new"], None,
                         st["table"], PAGE)
        pv.pv_segment_attention_prepared(ver.sizes, ver.plan, st["q"], st["k"], st["v"], st["out"], ver.workspace,
                                         st["lse"], 0.0, theta, st["table"], PAGE)
        logits = ver.judge_logits(st["hidden"], st["w2"])
        decision = ver.decide(logits, None, st["policy"])
        return [x for x in (st["out"], st["lse"], logits, decision) if x is not None]
    if case["kind"] == "segments":
        ver.segment_attention(st["q"], st["k"], st["v"], st["out"], st["lse"], rope_theta=theta)
    elif case["fp8"]:
        pv.pv_masked_attention_fp8kv(ver.sizes, ver.plan, st["q"], st["k"], st["v"], st["k_scale"], st["v_scale"],
                                     st["out"], ver.workspace, st["lse"], rope_theta=theta)
    else:
        ver.attention(st["q"], st["k"], st["v"], out=st["out"], lse=st["lse"], rope_theta=theta)
    readout = ver.first_reject(st["logits"], st["margin"])
    return [x for x in (st["out"], st["lse"], readout) if x is not None]


def work(case):
    """Both products over the visible (query, key) pairs; Q and O of the evaluated rows, K and V once."""
    problem = _problem(case)
    segments_only = case["kind"] != "pass"
    pairs = rows = 0
    for b in range(problem.batch):
        p, t, s = problem.prompt_len[b], problem.draft_len[b], problem.segment_len[b]
        c = p + t
        if not segments_only:
            pairs += c * (c + 1) // 2
            rows += c
        for x in problem.boundaries[b]:
            pairs += s * (p + x) + s * (s + 1) // 2
            rows += s
    n, d, hq, hkv = problem.total_tokens, case["head_dim"], case["q_heads"], case["kv_heads"]
    nbytes = rows * hq * d * 4 + n * hkv * d * 2 * (1 if case["fp8"] else 2)
    if case["lse"]:
        nbytes += rows * hq * 4
    flops = 4 * d * hq * pairs
    if case["kind"] == "judge":
        nbytes += problem.total_segments * HIDDEN * 2
        flops += 4 * HIDDEN * problem.total_segments
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Against the same pass in fp64 with the dense mask, the bf16 calls measured 1.5e-3 to 2.8e-3 of the
    result's norm and 6.5e-2 at most at one element (bf16 rounding of the rotated Q and K, of P and of
    O); the FP8 calls 2.0e-2 and 0.35 (P carries 3 mantissa bits, 2.7e-2 rms each).  Four times that,
    the FP8 norm within what two such roundings can differ by.  Verdicts and decisions are whole numbers
    taken in fp64: the same."""
    if case["fp8"]:
        return {"rel": 3e-2, "max": 0.9}
    return {"rel": 1e-2, "max": 0.25}
