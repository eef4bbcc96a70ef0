"""Lattices whose population buffer holds 2^32 words and more."""
import pytest
import torch

from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


def test_reset_clears_a_buffer_of_more_than_16_gib():
    """A 16400 x 16384 FP64 lattice in place (17.2 GB of populations) that has
    moved is at rest again after lbm_reset: without a force, u = 0 everywhere."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    nx, ny = 16400, 16384
    torch.cuda.empty_cache()
    say(f"reset {nx}x{ny} fp64 in place")
    s = lbm.Solver(nx, ny, "fp64", inplace=True, inplace_steps=1)
    s.set_material(0.4, 0.3)
    g = torch.ones(ny, nx, dtype=torch.float64, device="cuda")
    g[:, ::2] = -1.0
    s.set_body_force(g, g)
    s.step(3)
    zero = torch.zeros_like(g)
    s.set_body_force(zero, zero)
    assert all(bool((u != 0).any()) for u in s.displacement())
    s.reset()
    assert not any(bool((u != 0).any()) for u in s.displacement())
    s.close()
    del s, g, zero
    torch.cuda.empty_cache()
