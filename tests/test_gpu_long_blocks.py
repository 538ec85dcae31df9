"""The streaming kernel's two block sizes (one or two 32-query tiles per wave) in every pass it runs, on launches of which the rules of
csrc/flash_select.h send some to either (test_flash_select.py holds them to that): around the boundaries of its tiles, and with logits whose
maxima outgrow the rows' references, so that sub-tiles are formed again and the accumulators rescaled.

Bounds of the spiked inputs: entries reach hundreds; a weighted sum of bf16 rows with bf16-rounded weights, stored in bf16, is held to the
first-order analysis of these roundings (util.weighted_sum_bound), the relative norm to 1e-2."""
import math

import numpy as np
import pytest

from oracle import vmonarch_oracle as O
from paper_2601_22275_amd import synth
from tests import util as U

pytestmark = pytest.mark.gpu

# (d, with values): (tokens of a frame, frames) of updates in long blocks, whose last tiles lie on each of the four slots and hold 64, 1, 33 or
# 63 keys
_D128 = [(1024, 62), (1217, 50), (993, 63), (1023, 62), (1856, 32), (2049, 28), (1825, 32), (1855, 32),
         (1920, 32), (1857, 32), (1889, 32), (1919, 32), (1216, 50), (1153, 51), (1185, 51), (1215, 50)]
LONG_UPDATES = {
    (64, False): [(768, 129), (705, 129), (737, 129), (767, 129), (832, 110), (769, 110), (801, 110), (831, 110),
                  (640, 154), (833, 110), (609, 154), (639, 154), (704, 129), (641, 129), (673, 129), (703, 129)],
    (64, True): [(1024, 64), (1729, 36), (1249, 51), (1023, 64), (2624, 46), (2817, 42), (2849, 42), (2623, 46),
                 (2432, 51), (2625, 46), (2401, 51), (2431, 51), (1728, 36), (1921, 32), (1185, 101), (1727, 36)],
    (128, False): _D128, (128, True): _D128}
LONG_SPIKES = {(64, False): (705, 129), (64, True): (1247, 51), (128, False): (1217, 50), (128, True): (1217, 50)}
SHORT_SPIKES = (600, 1)
# heads, listed rows, keys of a head: exact rows
LONG_ROWS = [(51, 1025, 3970), (17, 257, 16001)]          # in one key range, in several
SHORT_ROWS = [(2, 130, 700), (2, 300, 9000)]              # the same
# frames, positions x heads: every pass of the temporal factor at d = 64 and the log-sum-exps at d = 128 in long blocks; in short ones
LONG_TEMPORAL, SHORT_TEMPORAL = (400, 512), (400, 6)
LONG_LAST = [(1249, 50), (8128, 8)]                       # the last sweep's pass at d = 128 in long blocks, the second at its limit
# heads, frames, tokens: the sink pass in long blocks at d = 64; in short ones
LONG_SINK, SHORT_SINK = (40, 26, 65), (2, 5, 161)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2601_22275_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    return torch, binding, torch.device("cuda:0")


def spiked(rng, nq, nk, d, spike):
    """Queries, keys and values whose logits hold a spike every 61 keys (or 16 in all), each `spike` higher than the last, which the
    queries answer with strengths of 0 to 9: with 72 the strongest rows' maxima grow by more than 2^56 from spike to spike, with 400
    by more than 2^192, past the exponents of float32."""
    q, k, v = (rng.normal(size=(n, d)) * s for n, s in ((nq, 0.8), (nk, 0.8), (nk, 1.0)))
    q[:, 0] = np.linspace(0.0, 9.0, nq)[rng.permutation(nq)]
    k[:, 0] = 0.0
    at = np.arange(17, nk, max(61, nk // 16))
    k[at, 0] = spike * np.arange(1, len(at) + 1)
    return [synth.f32_to_bf16_bits(x.astype(np.float32)) for x in (q, k, v)]


def check_rows(got, weights, x, what):
    ref = weights @ x
    ratio = np.abs(got - ref) / U.weighted_sum_bound(ref, weights @ np.abs(x))
    assert U.rel_l2(got, ref) <= U.BF16_REL_L2 and ratio.max() <= 1.0, (what, U.rel_l2(got, ref), float(ratio.max()))


def update_of_copies(env, frame, cR, frames, with_v):
    """One R-update of `frames` copies of a frame; every copy has to give the same bits.  The first one's aL, cL, y, lse."""
    torch, binding, dev = env
    b, d = frame[0].shape
    tq, tk, tv = (U.to_device([x], torch, dev).repeat(1, 1, frames, 1) for x in frame)
    tc = None if cR is None else torch.from_numpy(cR).to(dev).view(1, 1, b).repeat(1, 1, frames)
    out = binding.r_update_lse(tq, tc, tk, tv if with_v else None, frames, 1, b, 1.0 / math.sqrt(d), 0.1)
    first = []
    for x in out:
        if x is None:
            first.append(None)
            continue
        x = x.view(frames, b, -1)
        assert bool((x == x[:1]).all())
        first.append(x[0].float().cpu().numpy().astype(np.float64))
    return first


@pytest.mark.parametrize("d,with_v,b,frames", [(*k, *x) for k, v in LONG_UPDATES.items() for x in v])
def test_tile_boundaries(env, d, with_v, b, frames):
    """c_L and the log-sum-exp against 2^-8, what sums over weights rounded to bf16 would keep."""
    rng = np.random.default_rng(b + d)
    frame = [U.random_bits(rng, (b, d), 1.2, True) for _ in range(3)]
    cR = (0.2 + 2.0 * rng.random(b)).astype(np.float32)
    aL, cL, y, lse = update_of_copies(env, frame, cR, frames, with_v)
    q, k, v = (U.to_f64(x) for x in frame)
    z = q @ k.T / math.sqrt(d) / np.maximum(cR.astype(np.float64), 0.1)[:, None]
    R = O.softmax_rows(z)
    assert U.rel_l2(aL, R @ k) <= 4e-3 and U.max_abs(aL, R @ k) <= U.BF16_MAX_ABS
    assert U.max_abs(cL[:, 0], O.neg_entropy_rows(R)) <= 2.0 ** -8
    assert U.max_abs(lse[:, 0], np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)) <= 2.0 ** -8
    if with_v:
        assert U.rel_l2(y, R @ v) <= 4e-3 and U.max_abs(y, R @ v) <= U.BF16_MAX_ABS


@pytest.mark.parametrize("spike", [72.0, 400.0])
@pytest.mark.parametrize("with_v", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("blocks", ["long", "short"])
def test_moving_references_in_updates(env, blocks, d, with_v, spike):
    b, frames = LONG_SPIKES[d, with_v] if blocks == "long" else SHORT_SPIKES
    frame = spiked(np.random.default_rng(b + d), b, b, d, spike)
    aL, cL, y, lse = update_of_copies(env, frame, None, frames, with_v)
    q, k, v = (U.to_f64(x) for x in frame)
    z = q @ k.T / math.sqrt(d)
    R = O.softmax_rows(z)
    check_rows(aL, R, k, "aL")
    if with_v:
        check_rows(y, R, v, "y")
    # fp32 sums of sqrt(b) roundings, relative to a reference up to 96 binary orders (67 in natural units) away, and logits that are fp32 sums
    # of d products, log2(d) roundings, which move c_L by sum R |log R - c| times as much; four times (the logits' part: twice) these
    ref = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
    log_R, c, u = z - ref[:, None], O.neg_entropy_rows(R), 2.0 ** -24
    logits = 0.5 * math.log2(d) * np.abs(z).max(1)
    moved = logits * (R * np.abs(log_R - c[:, None])).sum(1)
    assert np.all(np.abs(cL[:, 0] - c) <= 4 * u * (moved + (67 + np.abs(c)) * math.sqrt(b)))
    assert np.all(np.abs(lse[:, 0] - ref) <= 4 * u * (logits + 67 + math.sqrt(b)))


@pytest.mark.parametrize("spike", [72.0, 400.0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,rows,N", LONG_ROWS + SHORT_ROWS)
@pytest.mark.parametrize("listed", [False, True])
def test_moving_references_in_exact_rows(env, heads, rows, N, d, listed, spike):
    torch, binding, dev = env
    rng = np.random.default_rng(rows + d)
    q, k, v = spiked(rng, N, N, d, spike)
    at = rng.permutation(N)[:rows] if listed else np.arange(rows)
    tq, tk, tv = (U.to_device([x], torch, dev).repeat(1, heads, 1, 1) for x in (q, k, v))
    out = torch.zeros_like(tq)
    if listed:
        binding.recompute_tokens(tq, tk, tv, 1, 1, N, out, torch.from_numpy(at.astype(np.int32)).to(dev))
    else:
        binding.recompute_rows(tq, tk, tv, 1, 1, N, out, 0, rows)
    assert bool((out == out[:, :1]).all())
    R = O.softmax_rows(U.to_f64(q)[at] @ U.to_f64(k).T / math.sqrt(d))
    check_rows(U.from_device(out)[0][at], R, U.to_f64(v), "rows")


@pytest.mark.parametrize("spike", [72.0, 400.0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,b", [LONG_SINK, SHORT_SINK, (2, 40, 700)])
def test_moving_references_in_the_sink_pass(env, heads, T, b, d, spike):
    torch, binding, dev = env
    N = T * b
    q, k, v = spiked(np.random.default_rng(b + d), N, b, d, spike)
    k, v = (np.concatenate([x, np.zeros((N - b, d), np.uint16)]) for x in (k, v))
    tq, tk, tv = (U.to_device([x], torch, dev).repeat(1, heads, 1, 1) for x in (q, k, v))
    out = binding.sink_average(tq, tk, tv, T, 1, b, torch.zeros_like(tq))
    assert bool((out == out[:, :1]).all())
    R = O.softmax_rows(U.to_f64(q) @ U.to_f64(k)[:b].T / math.sqrt(d))
    check_rows(2.0 * U.from_device(out)[0], R, U.to_f64(v)[:b], "sink")     # the average with zero: an exact half


@pytest.mark.parametrize("spike", [72.0, 400.0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,problems", [LONG_TEMPORAL, SHORT_TEMPORAL, LONG_LAST[0]])
def test_moving_references_in_the_temporal_factor(env, T, problems, d, spike):
    """Every position holds the same frames, every one has to give the same bits.  alpha_R and c_R are unnormalised sums of the rounded weights
    L: one rounding (2^-9 relative) of every term and, alpha_R, one of the sum."""
    torch, binding, dev = env
    rng = np.random.default_rng(T + d)
    Q, aL, Y = spiked(rng, T, T, d, spike)
    cL = (-3.0 * rng.random(T)).astype(np.float32)
    rep = lambda x: x.view(1, 1, T, 1, -1).expand(1, 1, T, problems, x.shape[-1]).reshape(1, 1, T * problems, -1)
    tq, ta, ty = (rep(U.to_device([x], torch, dev)) for x in (Q, aL, Y))
    tc = rep(torch.from_numpy(cL).to(dev).view(1, 1, T, 1)).view(1, 1, -1)
    s = 1.0 / math.sqrt(d)
    aR, cR = binding.l_update(tq, ta, tc, None, T, 1, problems, s)
    out = binding.l_update(tq, ta, tc, ty, T, 1, problems, s)
    for x in (aR, cR, out):
        x = x.view(T, problems, -1)
        assert bool((x == x[:, :1]).all())
    one = lambda x: x.view(T, problems, -1)[:, 0].float().cpu().numpy().astype(np.float64)
    Q, aL, Y = (U.to_f64(x) for x in (Q, aL, Y))
    L = O.softmax_rows(Q @ aL.T * s - cL.astype(np.float64)[None])
    check_rows(one(out), L, Y, "out")
    bound = lambda w: U.weighted_sum_bound(L.T @ w, L.T @ np.abs(w))
    # L itself: exp(u - lse), whose exponent carries the fp32 rounding of logits |u|: 2^-22 of the largest
    slack = 2.0 ** -22 * np.abs(Q @ aL.T * s).max() * (L.T @ np.abs(Q))
    assert np.all(np.abs(one(aR) - L.T @ Q) <= bound(Q) + slack)
    ones = np.ones((T, 1))
    assert np.all(np.abs(one(cR) - L.T @ ones) <= bound(ones) + 2.0 ** -22 * np.abs(Q @ aL.T * s).max() * (L.T @ ones))


@pytest.mark.parametrize("d", [64, 128])
def test_temporal_factor_at_its_longest(env, d):
    """As many frames as the key terms of a workgroup have room for: 64 rows of the first and the last position against the oracle."""
    torch, binding, dev = env
    T, problems = LONG_LAST[1]
    rng = np.random.default_rng(d)
    Q, aL, Y = (U.random_bits(rng, (T * problems, d), 1.2, True) for _ in range(3))
    cL = (-3.0 * rng.random(T * problems)).astype(np.float32)
    s = 1.0 / math.sqrt(d)
    out = U.from_device(binding.l_update(*(U.to_device([x], torch, dev) for x in (Q, aL)), torch.from_numpy(cL).to(dev).view(1, 1, -1),
                                         U.to_device([Y], torch, dev), T, 1, problems, s))[0].reshape(T, problems, d)
    rows = np.sort(rng.permutation(T)[:64])
    for i in (0, problems - 1):
        q, a, y = (U.to_f64(x).reshape(T, problems, d)[:, i] for x in (Q, aL, Y))
        L = O.softmax_rows(q[rows] @ a.T * s - cL.reshape(T, problems)[:, i].astype(np.float64)[None])
        assert U.rel_l2(out[rows, i], L @ y) <= 4e-3


@pytest.mark.parametrize("spike", [72.0, 400.0])
@pytest.mark.parametrize("d", [64, 128])
def test_moving_references_in_the_first_update_and_first_frame_together(env, d, spike):
    """A small call's first update and key ranges in one launch: the frames but the first keep the bits of the call without the first frame,
    whose update runs alone; the first frame is exact attention."""
    torch, binding, dev = env
    T, b, heads = 9, 257, 2
    rng = np.random.default_rng(d)
    q, k, v = spiked(rng, T * b, T * b, d, spike)
    tq, tk, tv = (U.to_device([x], torch, dev).repeat(1, heads, 1, 1) for x in (q, k, v))
    got = binding.attention(tq, tk, tv, T, 1, b, iters=2, recompute=1)
    rest = binding.attention(tq, tk, tv, T, 1, b, iters=2, recompute=0)
    assert torch.equal(got[:, :, b:].view(torch.uint8), rest[:, :, b:].view(torch.uint8))
    R = O.softmax_rows(U.to_f64(q)[:b] @ U.to_f64(k).T / math.sqrt(d))
    for h in range(heads):
        check_rows(U.from_device(got)[h, :b], R, U.to_f64(v), "first frame")
