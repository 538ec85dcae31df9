"""The calls this library's speed is judged on: attention over video clips and over general (m, b) splits of a
sequence, exact recomputation of chosen tokens, and the training pair of the blocked-softmax pass (forward with
its row statistics, backward), all through `paper_2601_22275_amd.binding`.

A case is a dict of plain values.  `kind` says which entry points run:

  attention   binding.attention: `iters` sweeps, then nothing / the exact first frame / the sink averaging
              (`recompute` 0 / 1 / 2)
  tokens      binding.recompute_tokens: exact attention of `rows` listed tokens of a finished output
  train       binding.r_update_lse, then binding.entropy_attention_bwd on its results (one block of training: O, the
              row statistics and all gradients); with_dH: a gradient also arrives through the entropy

Sizes: B x heads problems of T frames of Hs x Ws tokens with head dimension d, bf16 or f32.
"""
from __future__ import annotations

import math

import torch

from paper_2601_22275_amd import binding

_BASE = dict(B=1, heads=12, T=21, Hs=30, Ws=52, d=128, dtype="bf16")

F_BANDS = 8  # harmonics per coordinate of the positional features below


def listed():
    def case(name, kind, **kw):
        c = dict(_BASE)
        c.update(name=name, kind=kind, **kw)
        return c

    return [
        # the two ends of the paper's kernel benchmark (batch 1, 12 heads, d = 64, 32 blocks, 2 sweeps): 1024 tokens,
        # where the call is a chain of short launches, and 65,536 tokens
        case("attn-1k-d64", "attention", T=32, Hs=1, Ws=32, d=64, iters=2, recompute=0),
        case("attn-64k-d64", "attention", T=32, Hs=1, Ws=2048, d=64, iters=2, recompute=0),
        # a short low-resolution clip whose sizes are no multiple of anything, two samples in the batch, three sweeps
        case("attn-ragged-d64", "attention", B=2, heads=5, T=13, Hs=17, Ws=19, d=64, iters=3, recompute=1),
        # a 21-frame clip at 480p and at 720p, and a long clip at reduced resolution: two sweeps and the exact first frame,
        # what one attention layer of a video transformer asks for
        case("attn-480p", "attention", iters=2, recompute=1),
        case("attn-81-frames", "attention", T=81, Hs=28, Ws=52, iters=2, recompute=1),
        case("attn-720p", "attention", heads=40, Hs=45, Ws=80, iters=2, recompute=1),
        # the 480p clip with sink averaging in place of the exact first frame
        case("attn-480p-sink", "attention", iters=2, recompute=2),
        # many short blocks: 32,768 tokens as 512 blocks of 64, the far end of the computation-budget study
        case("attn-512x64", "attention", T=512, Hs=1, Ws=64, d=64, iters=2, recompute=0),
        # float32 tensors: a small clip as it is run to check a model in full precision
        case("attn-f32", "attention", heads=4, T=8, Hs=15, Ws=26, d=64, dtype="f32", iters=2, recompute=1),
        # exact attention of a thousand chosen tokens of the finished 480p clip
        case("tokens-480p", "tokens", rows=1000),
        # training on the 480p clip, the way the paper trains (no gradient through the entropy) ...
        case("train-480p", "train", with_dH=0, with_cR=0),
        # ... and on a ragged clip at d = 64 in a later sweep (rows scaled by c_R) with the entropy's gradient
        case("train-ragged-d64", "train", heads=10, T=9, Hs=23, Ws=41, d=64, with_dH=1, with_cR=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frame(rng, lo, hi):
    """Hs, Ws with lo <= Hs * Ws <= hi, spread over the logarithm, now and then one row (a split that is no video)."""
    while True:
        b = _log_int(rng, lo, hi)
        hs = 1 if rng.random() < 0.25 else max(1, int(round(math.sqrt(b * rng.uniform(0.4, 1.0)))))
        ws = max(1, int(round(b / hs)))
        if lo <= hs * ws <= hi:
            return hs, ws


def draw(rng):
    kind = rng.choices(["attention", "f32", "tokens", "train"], [5, 1, 1, 2])[0]
    largest = max(work(c)["flops"] for c in listed() if c["dtype"] == "bf16")
    largest_f32 = max(work(c)["flops"] for c in listed() if c["dtype"] == "f32")
    while True:
        c = dict(kind=kind, B=rng.choice([1, 1, 1, 2]), d=rng.choice([64, 128]), dtype="bf16")
        if kind == "attention":
            c["heads"] = _log_int(rng, 1, 40)
            c["T"] = _log_int(rng, 4, 512)
            # the whole range of frames for clips of up to 128 of them; beyond that the blocks are short
            c["Hs"], c["Ws"] = _frame(rng, 24, 3600 if c["T"] <= 128 else 160)
            c["iters"] = rng.choice([1, 2, 2, 3])
            c["recompute"] = rng.choice([0, 1, 1, 2])
        elif kind == "f32":
            c.update(kind="attention", dtype="f32", d=rng.choice([32, 64, 128]), heads=rng.randint(1, 4))
            c["T"] = _log_int(rng, 4, 32)
            c["Hs"], c["Ws"] = _frame(rng, 16, 512)
            c["iters"] = rng.choice([1, 2, 2, 3])
            c["recompute"] = rng.choice([0, 1, 1])
        elif kind == "tokens":
            c["heads"] = _log_int(rng, 2, 24)
            c["T"] = _log_int(rng, 4, 81)
            c["Hs"], c["Ws"] = _frame(rng, 100, 1560)
            c["rows"] = _log_int(rng, 8, 2000)
        else:
            c["heads"] = _log_int(rng, 1, 24)
            c["T"] = _log_int(rng, 2, 48)
            c["Hs"], c["Ws"] = _frame(rng, 40, 2400)
            c["with_dH"] = rng.randint(0, 1)
            c["with_cR"] = rng.randint(0, 1)
        n = c["T"] * c["Hs"] * c["Ws"]
        if kind == "tokens" and c["rows"] > n:
            continue
        if n < 64 or c["B"] * c["heads"] * n * c["d"] > 40 * 21 * 3600 * 128:
            continue
        if work(c)["flops"] > (largest_f32 if c["dtype"] == "f32" else largest):
            continue
        return c


def _video_tokens(case, gen, dev):
    """q, k, v [B, heads, N, d] float32 whose logits peak for tokens at nearby (frame, row, column): shared random
    projections of sines and cosines of the normalised coordinates, plus noise, scaled so that the logits
    q . k / sqrt(d) of random token pairs have a standard deviation of 3 (bf16), or left as they are (f32)."""
    bh, d = case["B"] * case["heads"], case["d"]
    ext = (case["T"], case["Hs"], case["Ws"])
    n = ext[0] * ext[1] * ext[2]
    coords = torch.meshgrid(*(torch.arange(e, device=dev, dtype=torch.float64) / e for e in ext), indexing="ij")
    phi = torch.stack([f(2.0 * math.pi * r * x.reshape(-1)) for x in coords for r in range(1, F_BANDS + 1)
                       for f in (torch.sin, torch.cos)], dim=1).float()
    pa, pb = (torch.randint(0, n, (4096,), generator=gen, device=dev) for _ in range(2))
    q, k, v = (torch.empty(bh, n, d, device=dev) for _ in range(3))
    for h in range(bh):
        w = torch.randn(2, phi.shape[1], d, generator=gen, device=dev) / math.sqrt(phi.shape[1])
        base = phi @ w[0]
        q[h] = torch.randn(n, d, generator=gen, device=dev) * 0.5 + base
        k[h] = torch.randn(n, d, generator=gen, device=dev) * 0.5 + base
        v[h] = torch.randn(n, d, generator=gen, device=dev) * 0.5 + phi @ w[1]
        if case["dtype"] == "bf16":
            gain = torch.sqrt(3.0 * math.sqrt(d) / (q[h, pa] * k[h, pb]).sum(1).std().clamp_min(1e-3))
            q[h] *= gain
            k[h] *= gain
    shape = (case["B"], case["heads"], n, d)
    return q.view(shape), k.view(shape), v.view(shape)


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    q, k, v = (x.to(dt) for x in _video_tokens(case, gen, dev))
    s = dict(case=case, q=q, k=k, v=v)
    n = q.shape[2]
    if case["kind"] == "tokens":
        s["out"] = torch.randn(q.shape, generator=gen, device=dev).to(dt)
        s["rows"] = torch.randperm(n, generator=gen, device=dev)[:case["rows"]].to(torch.int32)
    elif case["kind"] == "train":
        stat = (case["B"], case["heads"], n)
        s["dO"] = torch.randn(q.shape, generator=gen, device=dev).to(dt)
        s["dH"] = torch.randn(stat, generator=gen, device=dev) if case["with_dH"] else None
        s["cR"] = 0.3 + 1.5 * torch.rand(stat, generator=gen, device=dev) if case["with_cR"] else None
    return s


def run(state):
    c, q, k, v = state["case"], state["q"], state["k"], state["v"]
    size = (c["T"], c["Hs"], c["Ws"])
    if c["kind"] == "attention":
        return binding.attention(q, k, v, *size, iters=c["iters"], recompute=c["recompute"])
    if c["kind"] == "tokens":
        return binding.recompute_tokens(q, k, v, *size, state["out"], state["rows"])
    scale, cr_min = 1.0 / math.sqrt(c["d"]), 0.1
    aL, cL, y, lse = binding.r_update_lse(q, state["cR"], k, v, *size, scale, cr_min)
    dq, dk, dv = binding.entropy_attention_bwd(q, state["cR"], k, v, y, state["dO"], lse, -cL, state["dH"], *size,
                                               scale, cr_min)
    return dict(aL=aL, cL=cL, y=y, lse=lse, dq=dq, dk=dk, dv=dv)


def work(case):
    bh, T, b, d = case["B"] * case["heads"], case["T"], case["Hs"] * case["Ws"], case["d"]
    n = T * b
    tok = bh * n * d * (2 if case["dtype"] == "bf16" else 4)  # bytes of one token tensor
    stat = bh * n * 4                                         # ... of one float per token
    if case["kind"] == "attention":
        # per sweep: logits and R K inside the frames, logits and L^T Q (the last time R V and L y too) across them;
        # the exact first frame: b queries against n keys; the sink: n queries against b keys
        fl = case["iters"] * (4 * T * b * b * d + 4 * b * T * T * d) + 2 * T * b * b * d
        if case["recompute"]:
            fl += 4 * b * n * d
        return {"bytes": 4 * tok, "flops": bh * fl}
    if case["kind"] == "tokens":
        rows = case["rows"]
        listed_rows = bh * rows * d * (2 if case["dtype"] == "bf16" else 4)
        return {"bytes": 2 * tok + 2 * listed_rows + 4 * rows, "flops": bh * 4 * rows * n * d}
    # forward: three products (logits, R K, R V); backward: five (logits, dP, dV, dK, dQ)
    return {"bytes": 9 * tok + stat * (2 + case["with_dH"] + case["with_cR"]), "flops": bh * 16 * T * b * b * d}


def tolerance(case):
    """About four times the difference measured between these calls and the same arithmetic in float64 with the stored
    intermediates rounded where the data type rounds them, and between the library's kernel families (the same sums in
    another order): the largest relative 2-norm and element seen over the listed cases and 16 drawn ones."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}    # seen 5.6e-7 and 6e-6 (at most 2 sweeps, d <= 64)
    if case["kind"] == "attention":
        return {"rel": 1e-2, "max": 0.15}    # seen 2.6e-3 and 4e-2 (three sweeps)
    if case["kind"] == "tokens":
        # only the listed rows carry an error: the norm of the whole output dilutes it (seen 1.7e-4 at 1000 of 32,760 rows)
        share = case["rows"] / (case["T"] * case["Hs"] * case["Ws"])
        return {"rel": 4e-3 * math.sqrt(share), "max": 2e-2}
    # dQ and dK are small differences of large terms on sharp rows: seen 6.6e-3 and 0.33 of the root mean square on a
    # single element of dQ (dV and the forward results stay below 3e-3 and 0.07)
    return {"rel": 2.5e-2, "max": 0.9}
