"""c_L and the log-sum-exp of the R-update on every bf16 kernel that the default settings choose, with logits that share a
large part: both come from fp32 sums relative to the row's reference, so neither their digits nor the bf16 rounding of
the weights may show.  And rows without any finite logit.

Tolerance, u = 2^-24.  A logit z is an fp32 sum of exact products: its error is a few u |z|.  It moves the log-sum-exp by as
much, and c_L by sum_l R_l |log R_l - c_L| times as much.  The sums l and h of up to b terms carry sqrt(b) u, and h is taken
relative to a reference up to 64 binary orders (45 in natural units) away from the row's maximum.  Four times the sum of
these is allowed.  Weights rounded to bf16 in the sums, or a c_L formed as a difference of terms of the logits' size, miss it
by a factor of ten."""
import math

import numpy as np
import pytest

from paper_2601_22275_amd import synth
from tests import util as U
from tests.test_gpu_long_blocks import LONG_SPIKES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("common", [0.0, 300.0, 1000.0, 5000.0])
@pytest.mark.parametrize("d,b,frames,with_v", [
    (64, 40, 3, True), (64, 40, 3, False), (128, 40, 3, True), (128, 40, 3, False),  # a whole frame per workgroup
    (64, 300, 130, True), (64, 300, 130, False),                                     # one query tile per wave
    (64, 500, 2, True), (64, 500, 2, False), (128, 500, 2, True), (128, 500, 2, False),
    *((d, *LONG_SPIKES[d, v], v) for d, v in LONG_SPIKES),                           # two query tiles per wave
])
@pytest.mark.parametrize("spread", [0.3, 4.0])
def test_large_common_part(d, b, frames, with_v, common, spread):
    import torch
    from paper_2601_22275_amd import binding
    rng = np.random.default_rng(b + d)
    axis = np.where(rng.random(d) < 0.5, -1.0, 1.0) * math.sqrt(common / math.sqrt(d))
    noise = math.sqrt(spread) * d ** -0.125
    q, k, v = (synth.f32_to_bf16_bits((a + noise * rng.standard_normal((frames * b, d))).astype(np.float32))
               for a in (axis, axis, 0.0))
    dev = torch.device("cuda:0")
    tq, tk, tv = (U.to_device([x], torch, dev) for x in (q, k, v))
    s = 1.0 / math.sqrt(d)
    _, cL, _, lse = binding.r_update_lse(tq, None, tk, tv if with_v else None, frames, 1, b, s, 0.1)
    cL, lse = (U.from_device(x)[0].reshape(frames, b).astype(np.float64) for x in (cL, lse))
    u = 2.0 ** -24
    for j in sorted({0, frames // 2, frames - 1}):
        z = U.to_f64(q)[j * b:(j + 1) * b] @ U.to_f64(k)[j * b:(j + 1) * b].T * s
        ref = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
        log_R = z - ref[:, None]
        c = (np.exp(log_R) * log_R).sum(1)
        deviation = (np.exp(log_R) * np.abs(log_R - c[:, None])).sum(1)
        zmax = np.abs(z).max(1)
        assert np.all(np.abs(lse[j] - ref) <= 4 * u * (zmax + math.sqrt(b)))
        assert np.all(np.abs(cL[j] - c) <= 4 * u * (zmax * deviation + (45 + np.abs(c)) * math.sqrt(b)))


@pytest.mark.parametrize("d,b,frames", [(64, 40, 3), (128, 40, 3), (64, 300, 130), (64, 500, 2), (128, 500, 2)])
@pytest.mark.parametrize("with_v", [True, False])
def test_logits_of_minus_infinity(d, b, frames, with_v):
    """A frame whose logits all overflow to -inf gives zeros on every kernel, and the other frames what they give without it."""
    import torch
    from paper_2601_22275_amd import binding
    rng = np.random.default_rng(d + b)
    x = rng.standard_normal((3, frames * b, d)).astype(np.float32)
    x[0, :, 0] = 2.0
    dev = torch.device("cuda:0")
    results = []
    for key in (x[1, :b, 0].copy(), -3.3e38):
        x[1, :b, 0] = key
        tq, tk, tv = (U.to_device([synth.f32_to_bf16_bits(a)], torch, dev) for a in x)
        results.append(binding.r_update(tq, None, tk, tv if with_v else None, frames, 1, b, 1.0 / math.sqrt(d), 0.1))
    for finite, masked in zip(*results):
        if finite is None:
            continue
        assert torch.equal(finite[:, :, b:], masked[:, :, b:])
        if finite.dim() == 4:
            assert not masked[:, :, :b].any()
