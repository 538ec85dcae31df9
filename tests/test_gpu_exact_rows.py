"""Exact attention of chosen rows and the sink pass on both query-block sizes of the streaming kernel (128 and 256 rows): against
the CPU oracle and against the one-tile kernel (flash variant 0), which forms the same sums in another order.

Tolerance: the softmax weights and the result are rounded to bf16 (2^-9 relative each, random): sqrt(2) 2^-9 = 2.8e-3 in the relative
norm at most; 4e-3 against the oracle, 6e-3 between the kernels.  The sink pass averages with a value that is there already
and rounds once more: the same bounds."""
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


def _both(binding, call):
    got = call()
    binding.set_flash_variant(0)
    try:
        return U.from_device(got), U.from_device(call())
    finally:
        binding.set_flash_variant(2)


# heads x rows x keys: short blocks with key ranges, long blocks in one range, long blocks with ranges (and a last block of one row)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,rows,N", [(2, 130, 700), (51, 1025, 3970), (17, 257, 16001)])
def test_listed_rows(env, heads, rows, N, d):
    torch, binding, dev = env
    rng = np.random.default_rng(rows + d)
    q, k, v = (U.random_bits(rng, (heads, N, d), 1.5, True) for _ in range(3))
    tq, tk, tv = (U.to_device(list(x), torch, dev) for x in (q, k, v))
    listed = rng.permutation(N)[:rows].astype(np.int32)
    listed[[1, rows // 2]] = [-1, N]                      # entries that name no row are skipped
    tl = torch.from_numpy(listed).to(dev)
    base = torch.randn((1, heads, N, d), device=dev).bfloat16()
    got, one_tile = _both(binding, lambda: binding.recompute_tokens(tq, tk, tv, 1, 1, N, base.clone(), tl))
    rest = np.setdiff1d(np.arange(N), listed)
    valid = np.array([r for r in listed if 0 <= r < N])
    assert np.array_equal(got[:, rest], U.from_device(base)[:, rest])
    for h in (0, heads - 1):
        ref = O.softmax_attention(U.to_f64(q[h])[valid], U.to_f64(k[h]), U.to_f64(v[h]), 1.0 / math.sqrt(d))
        assert U.rel_l2(got[h][valid], ref) <= 4e-3
    assert U.rel_l2(got[:, valid], one_tile[:, valid]) <= 6e-3


@pytest.mark.parametrize("d", [64, 128])
def test_list_of_every_row(env, d):
    """A list as long as the head takes the kernel of one that is a row shorter: the rows both name get the same bits."""
    torch, binding, dev = env
    N, rng = 320, np.random.default_rng(d)
    tq, tk, tv = (U.to_device(list(U.random_bits(rng, (2, N, d), 1.5, True)), torch, dev) for _ in range(3))
    rows = torch.from_numpy(rng.permutation(N).astype(np.int32)).to(dev)
    zero = torch.zeros_like(tq)
    every, shorter = (binding.recompute_tokens(tq, tk, tv, 1, 1, N, zero.clone(), r) for r in (rows, rows[:-1].contiguous()))
    both = rows[:-1].long()
    assert torch.equal(every[:, :, both].view(torch.uint8), shorter[:, :, both].view(torch.uint8))


@pytest.mark.parametrize("d", [64, 128])
def test_merge_into_an_output_off_eight_bytes(env, d):
    """Several key ranges, merged into a tensor that starts two bytes into its storage: the bits of the aligned one, nothing beside it."""
    torch, binding, dev = env
    N, rows, rng = 9000, 300, np.random.default_rng(d)
    tq, tk, tv = (U.to_device(list(U.random_bits(rng, (2, N, d), 1.5, True)), torch, dev) for _ in range(3))
    ref = binding.recompute_rows(tq, tk, tv, 1, 1, N, torch.zeros_like(tq), 7, rows)
    storage = torch.full((tq.numel() + 8,), 3.0, dtype=tq.dtype, device=dev)
    out = storage[1:1 + tq.numel()].view(tq.shape)
    out.zero_()
    binding.recompute_rows(tq, tk, tv, 1, 1, N, out, 7, rows)
    assert out.data_ptr() % 8 == 2 and torch.equal(out, ref)
    assert bool((storage[:1] == 3.0).all()) and bool((storage[1 + tq.numel():] == 3.0).all())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,b", [(2, 5, 33), (40, 26, 65), (3, 2, 700)])
def test_sink_pass(env, heads, T, b, d):
    torch, binding, dev = env
    N = T * b
    rng = np.random.default_rng(T * b + d)
    q, k, v = (U.random_bits(rng, (heads, N, d), 1.5, True) for _ in range(3))
    tq, tk, tv = (U.to_device(list(x), torch, dev) for x in (q, k, v))
    base = torch.randn((1, heads, N, d), device=dev).bfloat16()
    got, one_tile = _both(binding, lambda: binding.sink_average(tq, tk, tv, T, 1, b, base.clone()))
    for h in (0, heads - 1):
        ref = O.softmax_attention(U.to_f64(q[h]), U.to_f64(k[h])[:b], U.to_f64(v[h])[:b], 1.0 / math.sqrt(d))
        assert U.rel_l2(got[h], (ref + U.from_device(base)[h]) / 2) <= 4e-3
    assert U.rel_l2(got, one_tile) <= 6e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,b", [(1, 5, 161), (2, 9, 257), (4, 13, 385), (12, 13, 300), (40, 30, 200)])
def test_first_frame_of_small_calls(env, heads, T, b, d):
    """A small call's first frame goes along with its first update (the last shape is too large for that): the other frames
    keep the bits of the call without it, the first frame agrees with the entry point of its own."""
    torch, binding, dev = env
    rng = np.random.default_rng(T * b + d)
    tq, tk, tv = (U.to_device(list(U.random_bits(rng, (heads, T * b, d), 1.5, True)), torch, dev) for _ in range(3))
    got = binding.attention(tq, tk, tv, T, 1, b, iters=2, recompute=1)
    rest = binding.attention(tq, tk, tv, T, 1, b, iters=2, recompute=0)
    assert torch.equal(got[:, :, b:].view(torch.uint8), rest[:, :, b:].view(torch.uint8))
    alone = binding.first_frame_attention(tq, tk, tv, T, 1, b, torch.zeros_like(tq))
    assert U.rel_l2(U.from_device(got[:, :, :b]), U.from_device(alone[:, :, :b])) <= 6e-3
    ref = O.softmax_attention(U.to_f64(tq[0, 0, :b].view(torch.uint16).cpu().numpy()), *(U.to_f64(x[0, 0].view(torch.uint16).cpu().numpy())
                              for x in (tk, tv)), 1.0 / math.sqrt(d))
    assert U.rel_l2(U.from_device(got)[0, :b], ref) <= 4e-3
