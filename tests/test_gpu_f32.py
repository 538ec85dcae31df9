"""The fp32 matrix-core kernels at the edges of their tiles (32 query rows, 32 keys, 1 / 2 / 4 waves per query tile, key
ranges of the recomputed rows, up to 32 frames), against the CPU oracle.

Tolerance: one fp32 rounding is 2^-24 = 6e-8; a sum of n terms carries about sqrt(n) of them (n <= 130 keys and 128
channels here), a logit of magnitude 10 another 10 of them through the exponential: about 2e-6 relative in the worst
direction, 1e-5 allowed."""
import math

import numpy as np
import pytest

from oracle import vmonarch_oracle as O
from tests import util as U

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2601_22275_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    return torch, binding, torch.device("cuda:0")


def _dev(torch, dev, arrs, misaligned=False):
    t = U.to_device(arrs, torch, dev)
    if not misaligned:
        return t
    # the same values on a 4-byte boundary: the call takes the plain-ALU kernels
    store = torch.empty(t.numel() + 1, dtype=t.dtype, device=dev)
    view = store[1:].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T,b,misaligned", [(2, 1, False), (3, 31, False), (2, 32, False), (1, 33, False), (2, 64, False),
                                            (1, 65, False), (1, 97, False), (1, 129, False), (700, 33, False), (1, 33, True)])
def test_r_update(env, T, b, d, misaligned):
    torch, binding, dev = env
    heads = 2
    rng = np.random.default_rng(31 * T + b + d)
    aR, K, V = ([U.random_bits(rng, (T * b, d), 1.0, False) for _ in range(heads)] for _ in range(3))
    cR = (0.03 + 2.5 * rng.random((heads, T * b))).astype(np.float32)
    s = 1.0 / math.sqrt(d)
    aL, cL, y, lse = binding.r_update_lse(_dev(torch, dev, aR, misaligned), torch.from_numpy(cR).to(dev).view(1, heads, -1),
                                          U.to_device(K, torch, dev), U.to_device(V, torch, dev), T, 1, b, s, 0.1)
    aL, cL, y, lse = (U.from_device(x) for x in (aL, cL, y, lse))
    for h in range(heads):
        c = cR[h].reshape(T, b).astype(np.float64)
        q3, k3, v3 = (U.to_f64(x[h]).reshape(T, b, d) for x in (aR, K, V))
        oaL, ocL, R = O.r_update(q3 * s, c, k3, 0.1)
        z = np.einsum("jid,jld->jil", q3 * s / np.maximum(c, 0.1)[:, :, None], k3)
        ref_lse = (np.log(np.exp(z - z.max(2, keepdims=True)).sum(2)) + z.max(2)).reshape(-1)
        assert U.rel_l2(aL[h], oaL.transpose(1, 0, 2).reshape(T * b, d)) <= TOL
        assert U.rel_l2(y[h], np.matmul(R, v3).reshape(T * b, d)) <= TOL
        assert U.max_abs(cL[h], ocL.T.reshape(-1)) <= TOL * max(1.0, np.abs(z).max())
        assert U.max_abs(lse[h], ref_lse) <= TOL * max(1.0, np.abs(z).max())


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T,b,iters,rec", [(32, 3, 2, 1), (31, 1, 2, 2), (9, 70, 1, 1), (33, 5, 2, 1), (20, 33, 3, 1)])
def test_attention(env, T, b, iters, rec, d):
    """T = 33: the plain-ALU temporal factor between matrix-core passes; 9 x 70 and 20 x 33: several key ranges."""
    torch, binding, dev = env
    data = U.structured_heads(T, 1, b, d, 17, 2, False)
    tq, tk, tv = (U.to_device([h[i] for h in data], torch, dev) for i in range(3))
    got = U.from_device(binding.attention(tq, tk, tv, T, 1, b, iters, rec))
    for h in range(2):
        q64, k64, v64 = (U.to_f64(x) for x in data[h])
        kw = dict(recompute=True) if rec == 1 else dict(sink_average=True)
        ref = O.monarch_attention(q64, k64, v64, T, b, iters, **kw)["O"].reshape(T * b, d)
        assert U.rel_l2(got[h], ref) <= TOL


@pytest.mark.parametrize("d", [32, 64, 128])
def test_listed_rows(env, d):
    """A list with both ends, a repeat and entries that are no rows of the head: those are skipped."""
    torch, binding, dev = env
    T, b = 5, 27
    data = U.structured_heads(T, 1, b, d, 18, 2, False)
    tq, tk, tv = (U.to_device([h[i] for h in data], torch, dev) for i in range(3))
    rows = [0, 134, 7, 7, -1, 135, 60] + list(range(90, 120))
    keep = torch.full_like(tq, 3.0)
    out = U.from_device(binding.recompute_tokens(tq, tk, tv, T, 1, b, keep, torch.tensor(rows, dtype=torch.int32, device=dev)))
    valid = sorted({r for r in rows if 0 <= r < T * b})
    rest = [r for r in range(T * b) if r not in valid]
    for h in range(2):
        q64, k64, v64 = (U.to_f64(x) for x in data[h])
        ref = O.softmax_attention(q64, k64, v64, 1.0 / math.sqrt(d))
        assert U.rel_l2(out[h][valid], ref[valid]) <= TOL
        assert np.all(out[h][rest] == 3.0)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T,b", [(3, 33), (7, 40), (29, 1)])
def test_infinite_value_in_the_last_row(env, T, b, d):
    """The rows that fill a tile past the last key or frame carry weight zero, and no infinity to multiply it with."""
    torch, binding, dev = env
    rng = np.random.default_rng(T + b + d)
    q, k, v = (U.random_bits(rng, (T * b, d), 0.5, False) for _ in range(3))
    v[b - 1::b, 3] = np.inf      # the last token of every frame ...
    v[(T - 1) * b:, 5] = -np.inf  # ... and every token of the last frame
    tq, tk, tv = (U.to_device([x], torch, dev) for x in (q, k, v))
    _, _, y = binding.r_update(tq, None, tk, tv, T, 1, b, 0.1, 0.1)
    out = binding.l_update(tq, tk, torch.zeros((1, 1, T * b), device=dev), tv, T, 1, b, 0.1)
    rows = binding.recompute_rows(tq, tk, tv, T, 1, b, torch.zeros_like(tq), 0, 2)
    y, out, rows = (U.from_device(x)[0] for x in (y, out, rows))
    frame, position = np.divmod(np.arange(T * b), b)
    assert np.all(np.isposinf(y[:, 3])) and np.all(np.isneginf(y[frame == T - 1, 5]))
    assert np.all(np.isposinf(out[position == b - 1, 3])) and np.all(np.isneginf(out[:, 5]))
    assert np.all(np.isposinf(rows[:2, 3])) and np.all(np.isneginf(rows[:2, 5]))
    rest = [c for c in range(d) if c not in (3, 5)]
    assert np.all(np.isfinite(y[:, rest])) and np.all(np.isfinite(out[:, rest])) and np.all(np.isfinite(rows[:2, rest]))
