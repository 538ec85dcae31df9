"""The four forms of the bf16 backward (with and without a gradient through the entropy, with and without row scales; with
neither the dK, dV pass takes its plain form) at the edges of its 32-row sub-tiles, 64-row tiles, the three-tile LDS rotation
and the owner blocks (128 rows at d = 64, 256 at d = 128), and with more blocks than fill the card once, against the CPU oracle on the forward results the library itself gave.

Tolerance: P and dS enter the products rounded to bf16 (2^-9 relative each), dS = P (dP - D) loses up to two more bits where
dP and D cancel (the inputs are random, dP - D is of dP's size in most elements), the results are rounded once more:
below 4 sqrt(2) 2^-9 = 1.1e-2 in the worst direction, 1e-2 in the relative norm."""
import math

import numpy as np
import pytest

from oracle import vmonarch_oracle as O
from tests import util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2601_22275_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    return torch, binding, torch.device("cuda:0")


@pytest.mark.parametrize("with_dh,with_cr", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("b", [2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 289, 384, 385, 513])
def test_backward_forms(env, b, d, with_dh, with_cr):
    torch, binding, dev = env
    T, rng = 2, np.random.default_rng(11 * b + d)
    Q, K, V, dO = (U.random_bits(rng, (T * b, d), 1.0, True) for _ in range(4))
    tq, tk, tv, tdo = (U.to_device([x], torch, dev) for x in (Q, K, V, dO))
    cR = (0.03 + 1.5 * rng.random(T * b)).astype(np.float32) if with_cr else None
    dH = rng.normal(size=T * b).astype(np.float32) if with_dh else None
    tcr, tdh = (None if x is None else torch.from_numpy(x).to(dev).view(1, 1, -1) for x in (cR, dH))
    s, cr_min = 1.0 / math.sqrt(d), 0.1
    _, cL, y, lse = binding.r_update_lse(tq, tcr, tk, tv, T, 1, b, s, cr_min)
    H = (-cL).contiguous()
    got = binding.entropy_attention_bwd(tq, tcr, tk, tv, y, tdo, lse, H, tdh, T, 1, b, s, cr_min)
    again = binding.entropy_attention_bwd(tq, tcr, tk, tv, y, tdo, lse, H, tdh, T, 1, b, s, cr_min)
    assert all(torch.equal(x, w) for x, w in zip(got, again))
    got = [U.from_device(x)[0].reshape(T, b, d) for x in got]
    q, k, v, do = (U.to_f64(x).reshape(T, b, d) for x in (Q, K, V, dO))
    o, l64, h64 = (U.from_device(x)[0].astype(np.float64).reshape(T, b, -1) for x in (y, lse, H))
    for j in range(T):
        c = np.ones(b) if cR is None else np.maximum(cR.reshape(T, b)[j].astype(np.float64), cr_min)
        dh = None if dH is None else dH.reshape(T, b)[j].astype(np.float64)
        ref = O.entropy_attention_backward(q[j], k[j], v[j], o[j], do[j], l64[j, :, 0], h64[j, :, 0], dh, s / c)
        for name, g, r in zip(("dq", "dk", "dv"), got, ref):
            assert U.rel_l2(g[j], r) <= 1e-2, name


@pytest.mark.parametrize("with_dh,with_cr", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("d", [64, 128])
def test_more_blocks_than_the_card_holds(env, d, with_dh, with_cr):
    """3 heads x 100 frames of 129 tokens: 600 owner blocks at d = 64, two of which share a compute unit.  The first, a middle and
    the last frame against the oracle, every frame against a second call."""
    torch, binding, dev = env
    T, b, heads, rng = 100, 129, 3, np.random.default_rng(d)
    Q, K, V, dO = ([U.random_bits(rng, (T * b, d), 1.0, True) for _ in range(heads)] for _ in range(4))
    tq, tk, tv, tdo = (U.to_device(x, torch, dev) for x in (Q, K, V, dO))
    cR = (0.03 + 1.5 * rng.random((heads, T * b))).astype(np.float32) if with_cr else None
    dH = rng.normal(size=(heads, T * b)).astype(np.float32) if with_dh else None
    tcr, tdh = (None if x is None else torch.from_numpy(x).to(dev).view(1, heads, -1) for x in (cR, dH))
    s, cr_min = 1.0 / math.sqrt(d), 0.1
    _, cL, y, lse = binding.r_update_lse(tq, tcr, tk, tv, T, 1, b, s, cr_min)
    H = (-cL).contiguous()
    got = binding.entropy_attention_bwd(tq, tcr, tk, tv, y, tdo, lse, H, tdh, T, 1, b, s, cr_min)
    again = binding.entropy_attention_bwd(tq, tcr, tk, tv, y, tdo, lse, H, tdh, T, 1, b, s, cr_min)
    assert all(torch.equal(x, w) for x, w in zip(got, again))
    got = [U.from_device(x) for x in got]
    y, lse, H = (U.from_device(x).astype(np.float64) for x in (y, lse, H))
    for h, j in ((0, 0), (1, 51), (2, T - 1)):
        rows = slice(j * b, (j + 1) * b)
        q, k, v, do = (U.to_f64(x[h][rows]) for x in (Q, K, V, dO))
        c = np.ones(b) if cR is None else np.maximum(cR[h][rows].astype(np.float64), cr_min)
        dh = None if dH is None else dH[h][rows].astype(np.float64)
        ref = O.entropy_attention_backward(q, k, v, y[h][rows], do, lse[h][rows], H[h][rows], dh, s / c)
        for name, g, r in zip(("dq", "dk", "dv"), got, ref):
            assert U.rel_l2(g[h][rows], r) <= 1e-2, name


@pytest.mark.parametrize("with_dh,with_cr", [(False, False), (True, True)])
def test_long_owner_blocks(env, with_dh, with_cr):
    """d = 128, 256 frames of 1200 tokens: a launch that takes owner blocks of 256 rows (smaller ones take 128).  Two frames repeated;
    every repeat bit-identical, one against the oracle."""
    torch, binding, dev = env
    b, d, frames, rng = 1200, 128, 256, np.random.default_rng(5)
    Q, K, V, dO = (U.random_bits(rng, (2 * b, d), 1.0, True) for _ in range(4))
    rep = lambda x: x.view(1, 1, 2, b, -1).repeat(1, 1, frames // 2, 1, 1).view(1, 1, frames * b, -1)
    tq, tk, tv, tdo = (rep(U.to_device([x], torch, dev)) for x in (Q, K, V, dO))
    cR = (0.3 + 1.5 * rng.random(2 * b)).astype(np.float32) if with_cr else None
    dH = rng.normal(size=2 * b).astype(np.float32) if with_dh else None
    tcr, tdh = (None if x is None else rep(torch.from_numpy(x).to(dev)).view(1, 1, -1) for x in (cR, dH))
    s, cr_min = 1.0 / math.sqrt(d), 0.1
    _, cL, y, lse = binding.r_update_lse(tq, tcr, tk, tv, frames, 1, b, s, cr_min)
    H = (-cL).contiguous()
    got = binding.entropy_attention_bwd(tq, tcr, tk, tv, y, tdo, lse, H, tdh, frames, 1, b, s, cr_min)
    for x in got:
        x = x.view(frames // 2, -1)
        assert bool((x == x[0]).all())
    got = [x.float().cpu().numpy().reshape(frames, b, d)[1] for x in got]
    q, k, v, do = (U.to_f64(x).reshape(2, b, d)[1] for x in (Q, K, V, dO))
    o, l64, h64 = (x.float().cpu().numpy().reshape(frames, b, -1)[1].astype(np.float64) for x in (y, lse, H))
    c = np.ones(b) if cR is None else np.maximum(cR[b:].astype(np.float64), cr_min)
    ref = O.entropy_attention_backward(q, k, v, o, do, l64[:, 0], h64[:, 0], None if dH is None else dH[b:].astype(np.float64), s / c)
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert U.rel_l2(g, r) <= 1e-2, name
