"""Lattices whose rows hold more bytes than a 32-bit offset reaches."""
import pytest
import torch

from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


def test_row_beyond_4_gib_equals_its_period():
    """A row of 2^30 + 896 FP32 sites (4 GiB per population) under a load of
    period 1118482 sites, which 2^30 is no multiple of, with free and with the
    default relaxation rates: after a few steps every period holds the displacement
    of a lattice of one period, bit for bit."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    p, k = 1118482, 960
    nx = p * k
    assert nx > 2 ** 30 and 2 ** 30 % p != 0
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 210 * 2 ** 30:
        pytest.skip("needs 210 GiB of GPU memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    half = torch.randint(-1000, 1000, (2, p // 2), generator=g, device="cuda").to(torch.float64) * 2.0 ** -30
    load = torch.cat([half, -half], dim=1)  # its mean is zero exactly

    def solver(m, reps):
        s = lbm.Solver(m, 1, "fp32")
        s.set_material(0.4, 0.3)
        s.set_body_force(*(load[c].repeat(reps).reshape(1, m) for c in (0, 1)))
        return s

    one, wide = solver(p, 1), solver(nx, k)
    for rates, n in (((0.3, 0.93, 0.9, 1.12), 5), ((1.0 / 3.0, 1.0, 1.0, 1.0), 2)):
        say(f"row of {nx} sites, rates {rates}")
        for s in (one, wide):
            s.reset()
            s.set_rates(*rates)
            s.step(n)
        for a, b in zip(wide.displacement(), one.displacement()):
            assert bool((a.reshape(k, p) == b.reshape(1, p)).all())
        del a, b
    one.close()
    wide.close()
    del one, wide, s
    torch.cuda.empty_cache()


def test_row_of_2_to_23_tiles():
    """One row of 2^29 FP32 sites through 64-wide tiles of 512 threads, a launch of
    2^32 threads if every tile had its workgroup: every period holds the displacement
    of a lattice of one period, bit for bit."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    p, k = 2 ** 20, 2 ** 9
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 120 * 2 ** 30:
        pytest.skip("needs 120 GiB of GPU memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    half = torch.randint(-1000, 1000, (2, p // 2), generator=g, device="cuda").to(torch.float64) * 2.0 ** -30
    load = torch.cat([half, -half], dim=1)  # its mean is zero exactly
    u = {}
    for m, reps in ((p, 1), (p * k, k)):
        s = lbm.Solver(m, 1, "fp32")
        s.set_material(0.4, 0.3)
        s.set_body_force(*(load[c].repeat(reps).reshape(1, m) for c in (0, 1)))
        s.set_time_blocking(8)
        s.set_fused_kernel("tile")
        say(f"row of {m} sites: {s.plain_launch()}")
        assert s.plain_launch()["kernel"] == "tile"
        s.step(8)
        u[m] = s.displacement()
        s.close()
        del s
        torch.cuda.empty_cache()
    for a, b in zip(u[p * k], u[p]):
        assert bool((a.reshape(k, p) == b.reshape(1, p)).all())
    u.clear()
    del a, b
    torch.cuda.empty_cache()
