"""The calls that programs make of this library, as cases to time and compare.

A case is one call of a public entry point of ``paper_1904_12380_amd`` on
fp32 GPU tensors, with the outputs allocated by the call as a program
usually leaves them to it:

    op "softmax"    softmax_fwd            [rows, cols] -> probabilities
    op "clip"       softmax_fwd_clip       the same, no clip (-inf)
    op "approx"     softmax_fwd_approx     the same, cheap exponential
    op "log"        softmax_log_fwd        log-probabilities
    op "nll"        softmax_nll_fwd        one loss per labelled row
    op "attention"  softmax_attention_fwd  softmax(Q K^T / sqrt(d)) V

``logits`` names the distribution of a row case's inputs:

    scores      N(0, 1): scaled dot products of attention
    classifier  N(0, 3^2), one entry of each row raised by 8
    vocab       N(0, 2^2), 5% of the entries masked to -1e4
    offset      N(0, 1) plus a per-row offset in U(-50, 50)
"""
from __future__ import annotations

import math

import torch

import paper_1904_12380_amd as sm

DEVICE = "cuda:0"
NEG_INF = float("-inf")


def _rows(name, op, rows, cols, logits):
    return {"name": name, "op": op, "rows": rows, "cols": cols, "logits": logits}


def _attention(name, batch, lq, lk, d, dv):
    return {"name": name, "op": "attention", "batch": batch, "lq": lq, "lk": lk, "d": d,
            "dv": dv}


def listed():
    return [
        # One request of the DAM model at batch 1: 9 turns x 50 query rows
        # over 50 keys.  The smallest call: launch and host time.
        _rows("dam_rows_450x50", "softmax", 450, 50, "scores"),
        # The same model at batch 256, the workload of its attention rows.
        _rows("dam_rows_115200x50", "softmax", 115200, 50, "scores"),
        # Training loss of a classifier over 1000 classes.
        _rows("classifier_nll_4096x1000", "nll", 4096, 1000, "classifier"),
        # Label log-probabilities of a sequence tagger: short rows of a
        # length that is no multiple of four.
        _rows("tagger_log_65536x130", "log", 65536, 130, "classifier"),
        # Vocabulary rows with masked entries, exact zeros for the masked
        # ones (no clip), of a power-of-two vocabulary.
        _rows("vocab_512x32768", "clip", 512, 32768, "vocab"),
        # Next-token probabilities over a vocabulary of an odd size.
        _rows("vocab_2048x30003", "softmax", 2048, 30003, "classifier"),
        # Language-model training loss, one large batch of tokens over an
        # odd vocabulary: the largest call.
        _rows("vocab_nll_16384x50001", "nll", 16384, 50001, "classifier"),
        # Long rows, the headline workload.
        _rows("longrow_64x262144", "softmax", 64, 262144, "offset"),
        # A few rows of millions of candidates (retrieval, sampling over a
        # whole catalogue).
        _rows("catalogue_8x4194304", "softmax", 8, 4194304, "offset"),
        # DAM attention, batch 256 x 9 turns.
        _attention("dam_attention_2304x50x50x200", 2304, 50, 50, 200, 200),
        # Attention heads over 64-token blocks.
        _attention("heads_attention_8192x64x64x64", 8192, 64, 64, 64, 64),
        # A few queries over a short sequence of 50-dimensional embeddings
        # (attention pooling; decoding with a short memory).
        _attention("pool_attention_16384x4x37x50", 16384, 4, 37, 50, 50),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["softmax", "softmax", "softmax", "clip", "approx", "log", "log", "nll",
                     "nll", "attention", "attention", "attention"])
    if op == "attention":
        lk = rng.randint(2, 64)
        lq = _log_uniform(rng, 1, 130)
        d = _log_uniform(rng, 16, 256)
        dv = d if rng.random() < 0.7 else _log_uniform(rng, 16, 256)
        if rng.random() < 0.6:  # heads are mostly whole multiples of 8
            d, dv = (max(8, 8 * round(x / 8)) for x in (d, dv))
        per_item = 4 * (lq + lk) * (d + dv)
        batch = max(1, _log_uniform(rng, 1 << 16, 1 << 28) // per_item)
        return {"op": op, "batch": batch, "lq": lq, "lk": lk, "d": d, "dv": dv}
    cols = _log_uniform(rng, 4, 1 << 22)
    if rng.random() < 0.5:  # half of the row lengths are whole 16-byte strips
        cols = max(4, 4 * round(cols / 4))
    elements = _log_uniform(rng, 1 << 15, 1 << 27)
    return {"op": op, "rows": max(1, elements // cols), "cols": cols,
            "logits": rng.choice(["scores", "classifier", "vocab", "offset"])}


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _logits(case, g):
    rows, cols, kind = case["rows"], case["cols"], case["logits"]
    x = torch.randn(rows, cols, device=DEVICE, generator=g)
    if kind == "classifier":
        x.mul_(3.0)
        hot = torch.randint(0, cols, (rows, 1), device=DEVICE, generator=g)
        x.scatter_add_(1, hot, torch.full((rows, 1), 8.0, device=DEVICE))
    elif kind == "vocab":
        x.mul_(2.0)
        x[torch.rand(rows, cols, device=DEVICE, generator=g) < 0.05] = -1.0e4
    elif kind == "offset":
        x.add_(100.0 * torch.rand(rows, 1, device=DEVICE, generator=g) - 50.0)
    return x


def _inputs(case, seed):
    g = _generator(seed)
    if case["op"] == "attention":
        b = case["batch"]
        return tuple(torch.randn(b, n, w, device=DEVICE, generator=g)
                     for n, w in ((case["lq"], case["d"]), (case["lk"], case["d"]),
                                  (case["lk"], case["dv"])))
    x = _logits(case, g)
    if case["op"] == "nll":
        return x, torch.randint(0, case["cols"], (case["rows"],), device=DEVICE, generator=g)
    return (x,)


def prepare(case, seed):
    return case["op"], _inputs(case, seed)


def run(state):
    op, t = state
    if op == "softmax":
        return sm.softmax_fwd(t[0])
    if op == "clip":
        return sm.softmax_fwd_clip(t[0], NEG_INF)
    if op == "approx":
        return sm.softmax_fwd_approx(t[0])
    if op == "log":
        return sm.softmax_log_fwd(t[0], NEG_INF)
    if op == "nll":
        return sm.softmax_nll_fwd(t[0], t[1], NEG_INF)
    return sm.softmax_attention_fwd(t[0], t[1], t[2])


def work(case):
    if case["op"] == "attention":
        b, lq, lk, d, dv = (case[k] for k in ("batch", "lq", "lk", "d", "dv"))
        return {"bytes": 4 * b * (lq * d + lk * d + lk * dv + lq * dv),
                "flops": 2 * b * lq * lk * (d + dv)}
    rows, cols = case["rows"], case["cols"]
    if case["op"] == "nll":
        return {"bytes": 4 * rows * cols + 12 * rows, "flops": 4 * rows * cols}
    return {"bytes": 8 * rows * cols, "flops": 5 * rows * cols}


def tolerance(case):
    # About four times the largest errors against 64 bits measured on the
    # listed cases and 60 drawn ones: rows rel 1.0e-7, max 5.4e-7 (fp32 sums
    # and exponentials); attention rel 4.1e-7, max 8.2e-6 (fp32 dot products).
    if case["op"] == "attention":
        return {"rel": 1.7e-6, "max": 3.3e-5}
    return {"rel": 4e-7, "max": 2.2e-6}


def _row_chunks(rows, cols):
    step = max(1, (1 << 26) // cols)
    return [(r, min(rows, r + step)) for r in range(0, rows, step)]


def exact(case, seed):
    t = _inputs(case, seed)
    if case["op"] == "attention":
        q, k, v = t
        scale = float(torch.tensor(1.0 / case["d"] ** 0.5, dtype=torch.float32))
        out = torch.empty(case["batch"], case["lq"], case["dv"], dtype=torch.float64,
                          device=DEVICE)
        per = case["lq"] * case["lk"] + (case["lq"] + case["lk"]) * (case["d"] + case["dv"])
        step = max(1, (1 << 26) // per)
        for b in range(0, case["batch"], step):
            kt = k[b:b + step].double().transpose(1, 2).contiguous()
            s = torch.bmm(q[b:b + step].double(), kt) * scale
            s = (s - s.amax(2, keepdim=True)).clamp(min=-64.0).exp()
            p = s / s.sum(2, keepdim=True)
            out[b:b + step] = torch.bmm(p, v[b:b + step].double())
        return out
    x = t[0]
    rows, cols = x.shape
    nll = case["op"] == "nll"
    out = torch.empty((rows,) if nll else (rows, cols), dtype=torch.float64, device=DEVICE)
    for a, b in _row_chunks(rows, cols):
        c = x[a:b].double()
        c = c - c.amax(1, keepdim=True)
        if case["op"] in ("softmax", "approx"):
            c = c.clamp(min=-64.0)
        s = c.exp().sum(1, keepdim=True)
        if nll:
            out[a:b] = (s.log() - c.gather(1, t[1][a:b, None]))[:, 0]
        elif case["op"] == "log":
            out[a:b] = c - s.log()
        else:
            out[a:b] = c.exp() / s
    return out
