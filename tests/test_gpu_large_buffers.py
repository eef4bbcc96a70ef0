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


def test_batch_of_more_than_2_to_22_tiles():
    """78 FP16 lattices of 7500 x 7500 (246 GB): a grid of 512-thread workgroups
    rounded up to the next power of two above their 4.3 M tiles would hold 2^32
    threads.  A checked chunk, which runs through the tiles, and single steps advance
    every lattice as a solver alone does."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    n, m = 7500, 78
    assert m * ((n + 63) // 64) * ((n + 15) // 16) > 2 ** 22
    torch.cuda.empty_cache()
    # the lattices, and the room for work-list items that the batch sizes by its arena
    arena = m * (lbm.Batch.slot_bytes(n, n, "fp16") + 2 * n * 14336) + (2 << 30)
    if torch.cuda.mem_get_info()[0] < arena + (12 << 30):
        pytest.skip("needs 260 GiB of GPU memory")
    x = torch.arange(n, dtype=torch.float64, device="cuda") * (2 * torch.pi / n)
    gx = 1e-6 * torch.sin(x)[:, None] * torch.cos(3 * x)[None, :]
    s = lbm.Solver(n, n, "fp16")
    s.set_material(0.4, 0.3)
    s.set_body_force(gx, gx)
    r = s.step_checked(8)  # rescales the half storage, which a batch does not
    s.reset()
    s.step(11)
    ref = s.displacement()
    s.close()
    b = lbm.Batch(m, arena)
    slots = [b.add(n, n, 0.4, 0.3, gx, gx, "fp16") for _ in range(m)]
    assert None not in slots
    say(f"{m} lattices {n}x{n} fp16, a checked chunk of eight, three single steps")
    b.step(8, check=True)
    rb, _ = b.residuals()
    assert all(abs(rb[i] - r) <= 1e-12 * r for i in slots)
    b.set_time_blocking(1)
    b.step(3)
    for i in slots:
        assert all(bool((a == e).all()) for a, e in zip(b.displacement(i), ref))
    b.close()
    del b, s, gx, x, ref
    torch.cuda.empty_cache()
