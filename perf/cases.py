"""Timed cases of the bucketed approximate top-k library: the calls that its users make, at the sizes they make them.

A case is one call of a public entry point on a matrix that already lies in GPU memory:
  call   "approx"      approx_topk(x, k, b, k_b)
         "contiguous"  approx_topk(x, k, b, k_b, assignment=ATK_CONTIGUOUS)
         "exact"       exact_topk(x, k)
  m, n   rows and row length;  dtype "f32" / "bf16";  k, b, k_b as in include/approx_topk.h
  data   "normal"  i.i.d. N(0, 1), the paper's own benchmark input (Appendix B.1)
         "scores"  q.K^T / sqrt(128), 64 queries to a head: attention scores (Section 4.2), many exact ties in bf16

Every output is a selection of input elements and their column indices, with ties decided, so outputs are compared
bit for bit.
"""
from __future__ import annotations

import math

import torch

import paper_2412_04358_amd as atk

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
_HEAD_DIM = 128   # of the attention scores
_QUERIES = 64     # rows that share a head's keys
_MAX_ELEMS = 1 << 27   # of a drawn matrix: what the largest listed exact selection reads


def _case(name, call, m, n, dtype, k, b=0, k_b=0, data="normal"):
    return dict(name=name, call=call, m=m, n=n, dtype=dtype, k=k, b=b, k_b=k_b, data=data)


def listed():
    return [
        # The smallest call anyone makes: four short rows, one survivor per bucket.  Launch and call latency.
        _case("small", "approx", 4, 4096, "f32", 64, 64, 1),
        # The paper's headline sweep (Figure 1 left) at b*k_b/k = 4: 128 rows, Stage 2 in the same launch.
        _case("headline", "approx", 128, 65536, "f32", 64, 256, 1),
        # The paper's k = n/4 sweep (Figure 1 right) with long queues and no Stage 2.
        _case("quarter_k", "approx", 128, 65536, "f32", 16384, 2048, 8),
        # Sparse attention over a batch of heads and queries (Section 4.2): short bf16 rows, the paper's k_b = 2 and
        # twice as many survivors as outputs for the recall, so every row has a large Stage 2.
        _case("attention", "approx", 2048, 8192, "bf16", 512, 512, 2, "scores"),
        # Sampling from the k most likely of a vocabulary's logits: rows that are no power of two.
        _case("vocabulary", "approx", 64, 128256, "bf16", 256, 512, 2),
        # Ranking the entities of a knowledge graph: very long rows of odd length.
        _case("entities", "approx", 128, 2653751, "bf16", 100, 512, 2),
        # Few buckets with long queues on very long rows: nearly every one of the true top 64 is found (recall 0.9999).
        _case("long_queues", "approx", 128, 1 << 20, "f32", 64, 128, 8),
        # k = n/16 with twice as many survivors: more candidates than one workgroup selects from.
        _case("many_candidates", "approx", 128, 65536, "f32", 4096, 4096, 2),
        # The contiguous bucket assignment that Appendix A.1 compares with.
        _case("contiguous", "contiguous", 128, 65536, "f32", 256, 512, 2),
        # The exact selection where the approximate one would be used: vocabulary logits, ...
        _case("exact_vocabulary", "exact", 64, 128256, "bf16", 256),
        # ... a batch of attention rows, ...
        _case("exact_attention", "exact", 2048, 8192, "bf16", 512, data="scores"),
        # ... and a quarter of very long rows: the most work that one call of the sweeps asks for.
        _case("exact_quarter_k", "exact", 128, 1 << 20, "f32", 1 << 18),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more call: batches of 1 to 2048 rows of 1024 to 2^21 elements, half of them powers of two, the rest odd lengths."""
    while True:
        m = _log_int(rng, 1, 2048)
        n = _log_int(rng, 1024, 1 << 21)
        style = rng.random()
        if style < 0.5:
            n = 1 << int(round(math.log2(n)))
        elif style < 0.75:
            n -= n % 8
        if rng.random() < 0.5:
            m = 1 << int(round(math.log2(m)))
        if m * n > _MAX_ELEMS or m * n < 8192:
            continue
        dtype = rng.choice(("f32", "bf16"))
        what = rng.random()
        call = "approx" if what < 0.6 else ("exact" if what < 0.9 else "contiguous")
        # small k as in sampling and ranking, or a fixed share of the row as in sparse attention and the k = n/4 sweep
        k = _log_int(rng, 16, 1024) if rng.random() < 0.6 else n // rng.choice((4, 8, 16))
        if k > n // 4:
            continue
        data = "scores" if dtype == "bf16" and n <= 16384 and rng.random() < 0.5 else "normal"
        c = dict(call=call, m=m, n=n, dtype=dtype, k=k, b=0, k_b=0, data=data)
        if call == "exact":
            return c
        k_b = rng.choice((1, 1, 1, 2, 2, 4, 8, 16))
        b = -(-k * rng.choice((1, 1, 2, 4, 8)) // k_b)
        if rng.random() < 0.5:
            b = 1 << max(0, math.ceil(math.log2(b)))
        if k_b > k or b > n or k_b > n // b or b * k_b > n // 2 or m * b * k_b > _MAX_ELEMS // 4:
            continue
        return dict(c, b=b, k_b=k_b)


def _input(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    m, n = case["m"], case["n"]
    if case["data"] == "scores":
        heads = -(-m // _QUERIES)
        q = torch.randn((heads, _QUERIES, _HEAD_DIM), generator=g, device="cuda")
        keys = torch.randn((heads, _HEAD_DIM, n), generator=g, device="cuda")
        x = (torch.matmul(q, keys) / math.sqrt(_HEAD_DIM)).reshape(heads * _QUERIES, n)[:m]
    else:
        x = torch.randn((m, n), generator=g, device="cuda")
    return x.to(_DTYPES[case["dtype"]]).contiguous()


def prepare(case, seed):
    return {"x": _input(case, seed), "call": case["call"], "k": case["k"], "b": case["b"], "k_b": case["k_b"]}


def run(state):
    if state["call"] == "exact":
        return atk.exact_topk(state["x"], state["k"])
    if state["call"] == "contiguous":
        return atk.approx_topk(state["x"], state["k"], state["b"], state["k_b"], assignment=atk.ATK_CONTIGUOUS)
    return atk.approx_topk(state["x"], state["k"], state["b"], state["k_b"])


def work(case):
    """Every element read once, k values and k 32-bit indices per row written once; comparisons only."""
    es = 4 if case["dtype"] == "f32" else 2
    return {"bytes": case["m"] * (case["n"] * es + case["k"] * (es + 4)), "flops": 0}


def tolerance(case):
    return "exact"


def _sorted_topk(vals, idx, k):
    """The k largest of each row of (value, index) pairs, largest first, the lower index first among equal values."""
    idx, order = idx.sort(dim=1)
    vals = vals.gather(1, order)
    vals, order = vals.sort(dim=1, descending=True, stable=True)
    return vals[:, :k].contiguous(), idx.gather(1, order)[:, :k].contiguous()


def _exact_rows(x, case):
    """The definition (Section 2) on a few rows, in float64, by sorting."""
    m, n = x.shape
    x = x.double()
    if case["call"] == "exact":
        vals, order = x.sort(dim=1, descending=True, stable=True)
        return vals[:, : case["k"]].contiguous(), order[:, : case["k"]].contiguous()
    k, b, k_b = case["k"], case["b"], case["k_b"]
    # bucket j as row j of a matrix of column indices, padded with n (an element below every other)
    if case["call"] == "contiguous":
        start = (torch.arange(b + 1, device=x.device) * n + b - 1) // b
        width = int((start[1:] - start[:-1]).max())
        at = start[:-1, None] + torch.arange(width, device=x.device)
        at = torch.where(at < start[1:, None], at, n)
    else:
        width = -(-n // b)
        at = torch.arange(b, device=x.device)[:, None] + b * torch.arange(width, device=x.device)
        at = torch.where(at < n, at, n)
    x = torch.cat([x, torch.full((m, 1), -math.inf, dtype=x.dtype, device=x.device)], dim=1)
    buckets = x[:, at.reshape(-1)].reshape(m * b, width)
    vals, order = buckets.sort(dim=1, descending=True, stable=True)
    rows = torch.arange(b, device=x.device).repeat(m)
    vals = vals[:, :k_b].reshape(m, b * k_b)
    idx = at[rows[:, None], order[:, :k_b]].reshape(m, b * k_b)
    return _sorted_topk(vals, idx, k) if b * k_b > k else (vals, idx)


def exact(case, seed):
    x = _input(case, seed)
    step = max(1, (1 << 25) // case["n"])
    parts = [_exact_rows(x[r: r + step], case) for r in range(0, case["m"], step)]
    return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts]).to(torch.int32)
