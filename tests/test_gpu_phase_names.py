"""Phase timing names what a phase holds: in small calls the first frame's key ranges go along with the first update."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,T,b,together", [(2, 9, 257, True), (40, 30, 200, False)])
def test_names(heads, T, b, together):
    import torch
    from paper_2601_22275_amd import binding
    q, k, v = (torch.randn((1, heads, T * b, 64), device="cuda").bfloat16() for _ in range(3))
    binding.set_phase_timing(True)
    try:
        binding.attention(q, k, v, T, 1, b, iters=2, recompute=1)
        names = [n for n, _ in binding.get_phase_timing()]
        binding.attention(q, k, v, T, 1, b, iters=2, recompute=0)
        without = [n for n, _ in binding.get_phase_timing()]
    finally:
        binding.set_phase_timing(False)
    sweeps = ["r_update", "l_update", "r_update_last", "l_update_last"]
    assert without == sweeps
    assert names == (["r_update+first_frame", *sweeps[1:], "first_frame_merge"] if together else [*sweeps, "first_frame"])
