"""The temporal factor over more than 128 frames in launches large enough to put two workgroups on every compute unit
(d = 64), against the CPU oracle at the first, a middle and the last position and against the small launch of those positions
alone, which runs the form with all registers.

Tolerance: the weights enter the products rounded to bf16 and the result is rounded to bf16 (2^-9 relative each, random):
sqrt(2) 2^-9 = 2.8e-3 in the relative norm at most, 4e-3 allowed against the oracle and 6e-3 between the two forms; c_R is a sum
of up to T rounded weights of sum c_R: 2^-9 relative, 2^-8 allowed."""
import numpy as np
import pytest

from oracle import vmonarch_oracle as O
from tests import util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [129, 192, 255, 257, 321, 513])
def test_large_launches(T):
    import torch
    from paper_2601_22275_amd import binding
    dev, b, d, heads, qs = torch.device("cuda:0"), 150, 64, 2, 0.125
    rng = np.random.default_rng(T)
    Q, aL, Y = ([U.random_bits(rng, (T * b, d), 1.5, True) for _ in range(heads)] for _ in range(3))
    cL = (-3.0 * rng.random((heads, T * b))).astype(np.float32)
    tq, taL, ty = (U.to_device(x, torch, dev) for x in (Q, aL, Y))
    tc = torch.from_numpy(cL).to(dev).view(1, heads, -1)
    pos = [0, 77, b - 1]
    pick = lambda x: x.view(1, heads, T, b, *x.shape[3:])[:, :, :, pos].contiguous().view(1, heads, T * 3, *x.shape[3:])
    aR, cR = binding.l_update(tq, taL, tc, None, T, 1, b, qs)
    out = binding.l_update(tq, taL, tc, ty, T, 1, b, qs)
    few = binding.l_update(pick(tq), pick(taL), pick(tc), None, T, 1, 3, qs)
    few_out = binding.l_update(pick(tq), pick(taL), pick(tc), pick(ty), T, 1, 3, qs)
    aR, cR, out = (U.from_device(pick(x)) for x in (aR, cR, out))
    few_aR, few_cR, few_out = (U.from_device(x) for x in (few[0], few[1], few_out))
    at = lambda x, h: U.to_f64(x[h]).reshape(T, b, -1)[:, pos].transpose(1, 0, 2)
    for h in range(heads):
        oaR, ocR, L = O.l_update(at(aL, h), cL[h].reshape(T, b)[:, pos].T.astype(np.float64), at(Q, h) * qs)
        assert U.rel_l2(aR[h] * qs, oaR.reshape(T * 3, d)) <= 4e-3
        assert U.rel_l2(cR[h], ocR.reshape(T * 3)) <= 2.0 ** -8
        assert U.rel_l2(out[h], np.matmul(L, at(Y, h)).transpose(1, 0, 2).reshape(T * 3, d)) <= 4e-3
        for got, ref in ((aR, few_aR), (out, few_out)):
            assert U.rel_l2(got[h], ref[h]) <= 6e-3
        assert U.rel_l2(cR[h], few_cR[h]) <= 2.0 ** -8


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [193, 256, 400])
def test_long_query_blocks(T, d):
    """Launches whose passes take query blocks of 256 rows (d = 128: the log-sum-exp pass), at the first, a middle and the last
    position against the oracle and the launch of those positions alone, which takes blocks of 128.  Bounds as above."""
    import torch
    from paper_2601_22275_amd import binding
    dev, b, heads, qs = torch.device("cuda:0"), 256, 2, d ** -0.5
    rng = np.random.default_rng(T + d)
    Q, aL, Y = ([U.random_bits(rng, (T * b, d), 1.5, True) for _ in range(heads)] for _ in range(3))
    cL = (-3.0 * rng.random((heads, T * b))).astype(np.float32)
    tq, taL, ty = (U.to_device(x, torch, dev) for x in (Q, aL, Y))
    tc = torch.from_numpy(cL).to(dev).view(1, heads, -1)
    pos = [0, 77, b - 1]
    pick = lambda x: x.view(1, heads, T, b, *x.shape[3:])[:, :, :, pos].contiguous().view(1, heads, T * 3, *x.shape[3:])
    large = (*binding.l_update(tq, taL, tc, None, T, 1, b, qs), binding.l_update(tq, taL, tc, ty, T, 1, b, qs))
    small = (*binding.l_update(pick(tq), pick(taL), pick(tc), None, T, 1, 3, qs),
             binding.l_update(pick(tq), pick(taL), pick(tc), pick(ty), T, 1, 3, qs))
    at = lambda x, h: U.to_f64(x[h]).reshape(T, b, -1)[:, pos].transpose(1, 0, 2)
    for (aR, cR, out) in ([U.from_device(pick(x)) for x in large], [U.from_device(x) for x in small]):
        for h in range(heads):
            oaR, ocR, L = O.l_update(at(aL, h), cL[h].reshape(T, b)[:, pos].T.astype(np.float64), at(Q, h) * qs)
            assert U.rel_l2(aR[h] * qs, oaR.reshape(T * 3, d)) <= 4e-3
            assert U.rel_l2(cR[h], ocR.reshape(T * 3)) <= 2.0 ** -8
            assert U.rel_l2(out[h], np.matmul(L, at(Y, h)).transpose(1, 0, 2).reshape(T * 3, d)) <= 4e-3
