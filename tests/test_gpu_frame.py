"""R-updates of short frames: the kernel that takes a whole frame per workgroup, at the edges of its 32-row tiles and on both sides of its
limits, against the CPU oracle and against the kernels of flash variant 0, which no such call takes by default and which form the same
sums in another order.

Tolerance: inputs, outputs and the softmax weights are bf16 (half an ulp is 2^-9 relative); alpha_L and y carry one rounding
of every weight and one of the result, both random: sqrt(2) 2^-9 = 2.8e-3 in the relative norm at most.  Against the
oracle 4e-3 is allowed, between the kernels 6e-3.  c_L and the log-sum-exp are held to 2^-8, what sums over weights
rounded to bf16 would keep (2^-9 relative, which the logarithm makes absolute, and as much again); the bound of the
float32 sums that they are is in test_gpu_row_statistics.py."""
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


def _inputs(T, b, d, seed):
    rng = np.random.default_rng(seed)
    aR, K, V = ([U.random_bits(rng, (T * b, d), 1.5, True) for _ in range(2)] for _ in range(3))
    return aR, K, V, (0.03 + 2.5 * rng.random((2, T * b))).astype(np.float32)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("b", [1, 2, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257])
@pytest.mark.parametrize("with_v", [True, False])
def test_r_update_of_short_frames(env, b, d, with_v):
    torch, binding, dev = env
    T, s = 3, 1.0 / math.sqrt(d)
    aR, K, V, cR = _inputs(T, b, d, 7 * b + d)
    tq, tk, tv = (U.to_device(x, torch, dev) for x in (aR, K, V))
    tc = torch.from_numpy(cR).to(dev).view(1, 2, -1)
    call = lambda: [None if x is None else U.from_device(x) for x in
                    binding.r_update_lse(tq, tc, tk, tv if with_v else None, T, 1, b, s, 0.1)]
    aL, cL, y, lse = call()
    binding.set_flash_variant(0)
    try:
        other = call()
    finally:
        binding.set_flash_variant(2)
    for h in range(2):
        c = np.maximum(cR[h].reshape(T, b).astype(np.float64), 0.1)
        q3, k3, v3 = (U.to_f64(x[h]).reshape(T, b, d) for x in (aR, K, V))
        oaL, ocL, R = O.r_update(q3 * s, c, k3, 0.1)
        z = np.einsum("jid,jld->jil", q3 * s / c[:, :, None], k3)
        ref_lse = (np.log(np.exp(z - z.max(2, keepdims=True)).sum(2)) + z.max(2)).reshape(-1)
        assert U.rel_l2(aL[h], oaL.transpose(1, 0, 2).reshape(T * b, d)) <= 4e-3
        assert U.rel_l2(aL[h], other[0][h]) <= 6e-3
        assert U.max_abs(cL[h], ocL.T.reshape(-1)) <= 2.0 ** -8
        assert U.max_abs(lse[h], ref_lse) <= 2.0 ** -8
        if with_v:
            assert U.rel_l2(y[h], np.matmul(R, v3).reshape(T * b, d)) <= 4e-3
            assert U.rel_l2(y[h], other[2][h]) <= 6e-3


@pytest.mark.parametrize("b", [257, 319, 320, 321, 352, 353, 383, 384, 385])
@pytest.mark.parametrize("with_v", [True, False])
def test_r_update_of_many_frames_beyond_the_whole_frame_kernel(env, b, with_v):
    """Frames of two to four query blocks of 128 rows of the streaming kernel, full ones and ragged ones: every frame against the
    kernels of variant 0, the first and the last one against the oracle."""
    torch, binding, dev = env
    T, d, s = 65, 64, 0.125
    aR, K, V, cR = _inputs(T, b, d, b)
    tq, tk, tv = (U.to_device(x, torch, dev) for x in (aR, K, V))
    tc = torch.from_numpy(cR).to(dev).view(1, 2, -1)
    call = lambda: [None if x is None else U.from_device(x) for x in
                    binding.r_update_lse(tq, tc, tk, tv if with_v else None, T, 1, b, s, 0.1)]
    aL, cL, y, lse = call()
    binding.set_flash_variant(0)
    try:
        other = call()
    finally:
        binding.set_flash_variant(2)
    for h in range(2):
        for j in range(T):
            rows = slice(j * b, (j + 1) * b)
            assert U.rel_l2(aL[h][rows], other[0][h][rows]) <= 6e-3
            assert not with_v or U.rel_l2(y[h][rows], other[2][h][rows]) <= 6e-3
            if j not in (0, T - 1):
                continue
            c = np.maximum(cR[h][rows].astype(np.float64), 0.1)[None]
            q3, k3, v3 = (U.to_f64(x[h][rows])[None] for x in (aR, K, V))
            oaL, ocL, R = O.r_update(q3 * s, c, k3, 0.1)
            z = (q3 * s / c[:, :, None] @ k3.transpose(0, 2, 1))[0]
            assert U.rel_l2(aL[h][rows], oaL[:, 0]) <= 4e-3
            assert U.max_abs(cL[h][rows], ocL.reshape(-1)) <= 2.0 ** -8
            assert U.max_abs(lse[h][rows], np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)) <= 2.0 ** -8
            if with_v:
                assert U.rel_l2(y[h][rows], np.matmul(R, v3)[0]) <= 4e-3


@pytest.mark.parametrize("d", [64, 128])
def test_many_frames_and_no_row_scale(env, d):
    """More frames than compute units, c_R absent, first and last frame against the oracle; a second call gives the same bits."""
    torch, binding, dev = env
    T, b, s = 700, 40, 1.0 / math.sqrt(d)
    aR, K, V, _ = _inputs(T, b, d, 5)
    tq, tk, tv = (U.to_device(x, torch, dev) for x in (aR, K, V))
    first = binding.r_update(tq, None, tk, tv, T, 1, b, s, 0.1)
    again = binding.r_update(tq, None, tk, tv, T, 1, b, s, 0.1)
    assert all(torch.equal(x, w) for x, w in zip(first, again))
    aL, cL, y = (U.from_device(x) for x in first)
    for h in range(2):
        for j in (0, T - 1):
            rows = slice(j * b, (j + 1) * b)
            q3, k3, v3 = (U.to_f64(x[h][rows])[None] for x in (aR, K, V))
            oaL, ocL, R = O.r_update(q3 * s, np.ones((1, b)), k3, 0.1)
            assert U.rel_l2(aL[h][rows], oaL[:, 0]) <= 4e-3
            assert U.max_abs(cL[h][rows], ocL.reshape(-1)) <= 2.0 ** -8
            assert U.rel_l2(y[h][rows], np.matmul(R, v3)[0]) <= 4e-3


@pytest.mark.parametrize("d,b,frames", [(64, 256, 512), (64, 260, 16), (64, 449, 256), (128, 161, 8), (128, 193, 300), (128, 1290, 256), (128, 1281, 16)])
@pytest.mark.parametrize("with_v", [False, True])
def test_query_blocks_of_the_streaming_kernel(env, d, b, frames, with_v):
    """Updates take query blocks of 128 or of 256 rows by the size of the launch (test_gpu_long_blocks.py drives the long ones): the same two
    frames in launches from a few blocks to several rounds, against the oracle (bounds as above), every repeat bit-identical."""
    torch, binding, dev = env
    s = 1.0 / math.sqrt(d)
    aR, K, V, cR = _inputs(1, b, d, 11 * b + d)
    tq, tk, tv = (U.to_device(x, torch, dev).reshape(1, 2, b, d).repeat(1, frames // 2, 1, 1).view(1, 1, -1, d) for x in (aR, K, V))
    tc = torch.from_numpy(cR).to(dev).view(1, 2, b).repeat(1, frames // 2, 1).view(1, 1, -1)
    aL, cL, y, lse = binding.r_update_lse(tq, tc, tk, tv if with_v else None, frames, 1, b, s, 0.1)
    got = [x.view(frames // 2, -1) for x in ((aL, cL, lse, y) if with_v else (aL, cL, lse))]
    for x in got:
        assert bool((x == x[0]).all())
    gaL = U.from_device(got[0][0].view(1, 1, 2 * b, d))[0].reshape(2, b, d)
    gcL = got[1][0].cpu().numpy().reshape(2, b)
    for h in range(2):
        c = np.maximum(cR[h].reshape(1, b).astype(np.float64), 0.1)
        q3, k3 = (U.to_f64(x[h]).reshape(1, b, d) for x in (aR, K))
        oaL, ocL, R = O.r_update(q3 * s, c, k3, 0.1)
        assert U.rel_l2(gaL[h], oaL[:, 0]) <= 4e-3
        if with_v:
            gy = U.from_device(got[3][0].view(1, 1, 2 * b, d))[0].reshape(2, b, d)[h]
            assert U.rel_l2(gy, R[0] @ U.to_f64(V[h]).reshape(b, d)) <= 4e-3
        assert U.max_abs(gcL[h], ocL.reshape(-1)) <= 2.0 ** -8
