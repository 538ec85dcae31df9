"""The references of the streaming kernel's running sums (flash2.hip): they stay at the rows' maxima, so that c_L keeps its digits and
values near the bottom of bf16's range keep theirs."""
import math

import numpy as np
import pytest

from paper_2601_22275_amd import synth
from tests import util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2601_22275_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    return torch, binding, torch.device("cuda:0")


@pytest.mark.parametrize("deviation", [1.0, 3.0])
@pytest.mark.parametrize("d,b,frames", [(64, 300, 130), (64, 700, 2), (64, 1000, 64), (128, 200, 130), (128, 700, 2), (128, 1000, 64)])
@pytest.mark.parametrize("with_v", [False, True])
def test_c_L_of_ordinary_rows(env, d, b, frames, with_v, deviation):
    """Root mean square of c_L's error over the rows of two frames, u = 2^-24: c_L = h / l - log l with fp32 sums of 16 terms and then
    b / 32 partial sums: n = 16 + b / 32 roundings of at most u relative, uniform and so u / sqrt(3) each, on sums that grow to h and l: n / 3 of
    them count fully, 0.25 u sqrt(n) with a mantissa's mean.  With the reference at the maximum of a row whose logits are of this deviation,
    1 <= l and |h / l| <= |c| + log l: 2 |c| + 4 covers both.  The fp32 rounding of the logits adds u / 2 |z| times sum R |log R - c|.  References
    2^64 above the maxima miss it by a factor of 2.5 and more."""
    torch, binding, dev = env
    rng = np.random.default_rng(b + d)
    q, k = (synth.f32_to_bf16_bits((math.sqrt(deviation) * rng.standard_normal((frames * b, d))).astype(np.float32)) for _ in range(2))
    tq, tk = (U.to_device([x], torch, dev) for x in (q, k))
    s = 1.0 / math.sqrt(d)
    _, cL, _ = binding.r_update(tq, None, tk, tk if with_v else None, frames, 1, b, s, 0.1)
    cL = U.from_device(cL)[0].reshape(frames, b).astype(np.float64)
    error, bound = [], []
    u = 2.0 ** -24
    for j in (0, frames - 1):
        z = U.to_f64(q)[j * b:(j + 1) * b] @ U.to_f64(k)[j * b:(j + 1) * b].T * s
        log_R = z - z.max(1, keepdims=True)
        log_R -= np.log(np.exp(log_R).sum(1, keepdims=True))
        c = (np.exp(log_R) * log_R).sum(1)
        spread = (np.exp(log_R) * np.abs(log_R - c[:, None])).sum(1)
        error.append(cL[j] - c)
        bound.append(0.25 * u * math.sqrt(16 + b / 32) * (2 * np.abs(c) + 4) + 0.5 * u * np.abs(z).max(1) * spread)
    rms = lambda x: float(np.sqrt(np.mean(np.square(x))))
    print(f"c_L d={d} b={b} x {frames} deviation {deviation}: rms error {rms(error):.2e}, bound {rms(bound):.2e}")
    assert rms(error) <= rms(bound)


@pytest.mark.parametrize("deviation", [20.0, 40.0])
@pytest.mark.parametrize("d,b,frames", [(64, 300, 130), (64, 1560, 2), (64, 1000, 64), (128, 200, 130), (128, 1560, 2), (128, 1100, 100)])
@pytest.mark.parametrize("with_v", [False, True])
def test_c_L_of_sharp_rows(env, d, b, frames, with_v, deviation):
    """Rows of few heavy keys, whose references have headroom and move: every element within four times the rounding of these keys' t, up to 96
    binary orders (67 in natural units) from the reference, and of the logits (log2(d) / 2 roundings), which move c_L by sum R |log R - c|
    times as much."""
    torch, binding, dev = env
    rng = np.random.default_rng(b + d)
    q, k = (synth.f32_to_bf16_bits((math.sqrt(deviation) * rng.standard_normal((frames * b, d))).astype(np.float32)) for _ in range(2))
    tq, tk = (U.to_device([x], torch, dev) for x in (q, k))
    s = 1.0 / math.sqrt(d)
    _, cL, _ = binding.r_update(tq, None, tk, tk if with_v else None, frames, 1, b, s, 0.1)
    cL = U.from_device(cL)[0].reshape(frames, b).astype(np.float64)
    u = 2.0 ** -24
    for j in (0, frames - 1):
        z = U.to_f64(q)[j * b:(j + 1) * b] @ U.to_f64(k)[j * b:(j + 1) * b].T * s
        log_R = z - z.max(1, keepdims=True)
        log_R -= np.log(np.exp(log_R).sum(1, keepdims=True))
        c = (np.exp(log_R) * log_R).sum(1)
        spread = (np.exp(log_R) * np.abs(log_R - c[:, None])).sum(1)
        assert np.all(np.abs(cL[j] - c) <= 4 * u * (67 + np.abs(c) + 0.5 * math.log2(d) * np.abs(z).max(1) * spread))


@pytest.mark.parametrize("exponent,deviation", [(-90, 2.0), (-110, 2.0), (-60, 40.0), (77, 40.0), (95, 2.0)])
@pytest.mark.parametrize("d", [64, 128])
def test_values_near_the_ends_of_the_range(env, d, exponent, deviation):
    """Values of the size 2^exponent through every pass that multiplies values, in ordinary rows and in sharp ones, whose weights grow to
    many orders above one: the same relative error as at size one (weights and result rounded to bf16, sqrt(2) 2^-9; 4e-3 allowed)."""
    torch, binding, dev = env
    rng = np.random.default_rng(d)
    T, b, s = 5, 400, 1.0 / math.sqrt(d)
    N = T * b
    q, k, v = (U.random_bits(rng, (N, d), scale, True) for scale in (math.sqrt(deviation), math.sqrt(deviation), 1.5))
    v = synth.f32_to_bf16_bits((U.to_f64(v) * 2.0 ** exponent).astype(np.float32))
    tq, tk, tv = (U.to_device([x], torch, dev) for x in (q, k, v))
    q, k, v = (U.to_f64(x) for x in (q, k, v))

    def attend(q, k, v):
        z = q @ k.swapaxes(-1, -2) * s
        p = np.exp(z - z.max(-1, keepdims=True))
        return p / p.sum(-1, keepdims=True) @ v

    rows = rng.permutation(N)[:300]
    zero = torch.zeros_like(tq)
    frames = lambda x: x.reshape(T, b, d)
    got = {
        "first frame": (binding.first_frame_attention(tq, tk, tv, T, 1, b, zero.clone()), lambda o: o[:b], attend(q[:b], k, v)),
        "row list": (binding.recompute_tokens(tq, tk, tv, T, 1, b, zero.clone(), torch.from_numpy(rows.astype(np.int32)).to(dev)),
                     lambda o: o[rows], attend(q[rows], k, v)),
        "sink": (binding.sink_average(tq, tk, tv, T, 1, b, zero.clone()), lambda o: 2 * o, attend(q, k[:b], v[:b])),
        "R-update": (binding.r_update(tq, None, tk, tv, T, 1, b, s, 0.1)[2], frames, attend(frames(q), frames(k), frames(v))),
        "temporal": (binding.l_update(tq, tk, torch.zeros((1, 1, N), device=dev), tv, b, 1, T, s),
                     lambda o: o.reshape(b, T, d).swapaxes(0, 1), attend(*(x.reshape(b, T, d).swapaxes(0, 1) for x in (q, k, v)))),
    }
    for name, (out, pick, ref) in got.items():
        assert U.rel_l2(pick(U.from_device(out)[0].astype(np.float64)) * 2.0 ** -exponent, ref * 2.0 ** -exponent) <= 4e-3, name
