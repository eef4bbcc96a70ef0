"""Wavefront launches that only some options reach (free relaxation rates, in
place at twelve steps, the default rule's smallest lattices), against single
steps bit for bit: every level is rounded as a store would round it, so no
tolerance.  Each case asserts that the wavefront is what runs."""
import numpy as np
import pytest

from gpu_common import dev, host, need_gpu, say
from paper_2208_14870_amd import problem as P

pytestmark = pytest.mark.gpu

RATES = (0.3, 0.93, 0.9, 1.12)


def _states(nx, ny, prec, steps, shape=None, want=None, rates=None, sr=False, inplace=False):
    """Populations after each of `steps` (cumulative); shape(solver) sets the
    launch shape, want: (depth, columns per lane) of the wavefront."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    rng = np.random.default_rng(nx * 31 + ny)
    f0 = rng.standard_normal((8, ny, nx))
    g = rng.standard_normal((2, ny, nx)) * 1e-2
    g -= g.mean(axis=(1, 2), keepdims=True)
    mat = P.Material.from_shear_poisson(0.9, 0.3)
    s = lbm.Solver(nx, ny, prec, inplace=inplace)
    if rates:
        s.set_rates(*rates)
    s.set_material(mat.lame_lambda, mat.lame_mu)
    if sr:
        s.set_stochastic_rounding(True, 7)
    s.set_body_force(dev(g[0]), dev(g[1]))
    s.set_populations(dev(f0))
    if shape:
        shape(s)
    if want:
        p = s.plain_launch()
        assert p["kernel"] == "wavefront", p
        assert (p["steps_per_launch"], p["columns_per_lane"]) == want, p
    out = []
    for n in steps:
        s.step(n)
        out.append(host(s.populations()))
    s.close()
    return out


def _same(nx, ny, prec, steps, shape=None, want=None, **kw):
    say(f"wavefront {prec} {nx}x{ny} {want} {kw}")
    got = _states(nx, ny, prec, steps, shape, want, **kw)
    kw.pop("inplace", None)
    ref = _states(nx, ny, prec, steps, lambda s: s.set_time_blocking(1), **kw)
    for n, a, b in zip(np.cumsum(steps), got, ref):
        np.testing.assert_array_equal(a, b, err_msg=f"after {n} steps")


# below one strip, at and one beyond a strip's output columns (wide and narrow),
# odd and even, short and tall; segments shorter and longer than the lattice
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,rows", [(1, 1, 4), (3, 2, 1), (20, 21, 7), (97, 31, 16), (106, 12, 5),
                                        (109, 50, 64), (250, 13, 13), (122, 40, 9)])
def test_general_rates_through_the_chosen_wavefront(prec, nx, ny, rows):
    """Free relaxation rates at every chosen depth: full launches and every
    remainder."""
    for depth in range(2, 9):
        v = 2 if prec != "fp64" and nx % 2 == 0 and depth <= 4 else 1

        def shape(s):
            s.set_time_blocking(depth)
            s.set_fused_kernel("wavefront", rows)
        _same(nx, ny, prec, (depth, 2 * depth + depth // 2, 3), shape, (depth, v), rates=RATES)


# just past the small-lattice rule: strips of 98 (108 for half storage) columns
# filled exactly, one beyond, and ragged
@pytest.mark.parametrize("prec,nx,ny", [("fp64", 490, 420), ("fp64", 491, 419), ("fp32", 490, 420),
                                        ("fp32", 491, 419), ("fp16", 540, 400), ("fp16", 541, 401)])
def test_general_rates_at_the_default_depth(prec, nx, ny):
    """Free relaxation rates at the library's own depth: full launches, and the
    remainders of one and of two launches."""
    deep = 8 if prec == "fp16" else 12
    _same(nx, ny, prec, (deep, 9, 11, 2 * deep + 10, 7), None, (deep, 1), rates=RATES)


# sizes whose longer segments leave the room for twelve steps: odd and even
# widths, one and two columns per lane, heights that the segments do not divide
@pytest.mark.parametrize("prec,nx,ny,v", [("fp64", 1000, 1000, 1), ("fp64", 701, 1536, 1),
                                          ("fp32", 1001, 1000, 1), ("fp32", 2048, 1536, 2)])
def test_in_place_at_twelve_steps(prec, nx, ny, v):
    """In place at the default depth, from both layouts, with remainders of every
    kind."""
    _same(nx, ny, prec, (13, 12, 23, 24, 35, 1, 12), None, (12, v), inplace=True)


# strips of one wave: widths at its output columns (40 at twelve steps, 48 at
# eight), one beyond, and far below; by default, with free rates, in place (odd
# widths, or FP64) and with stochastic rounding
NARROW = [("fp64", 40, 5000, 12, 256, ""), ("fp64", 48, 4000, 8, 192, ""), ("fp64", 3, 90001, 12, 256, ""),
          ("fp32", 39, 10007, 12, 256, ""), ("fp32", 40, 9001, 12, 256, ""), ("fp32", 47, 9000, 8, 192, ""),
          ("fp32", 1, 400003, 12, 256, ""), ("fp16", 48, 30011, 8, 256, ""), ("fp16", 5, 300001, 8, 256, ""),
          ("fp64", 40, 5000, 12, 256, "rates"), ("fp64", 48, 4000, 8, 192, "rates"),
          ("fp32", 8, 50000, 12, 256, "rates"), ("fp32", 47, 9000, 8, 192, "rates"),
          ("fp16", 48, 9001, 8, 256, "rates"), ("fp16", 20, 20011, 8, 256, "rates"),
          ("fp64", 48, 4000, 8, 192, "in place"), ("fp64", 3, 9001, 8, 192, "in place"),
          ("fp32", 39, 10007, 8, 192, "in place"), ("fp16", 48, 3001, 8, 256, "in place"),
          ("fp16", 47, 50000, 8, 256, "stochastic")]


@pytest.mark.parametrize("prec,nx,ny,depth,threads,kind", NARROW)
def test_narrow_lattices_take_strips_of_one_wave(prec, nx, ny, depth, threads, kind):
    """Lattices no wider than a strip of one wave: full launches and every
    remainder."""
    def shape(s):
        p = s.plain_launch()
        assert (p["kernel"], p["steps_per_launch"], p["threads"]) == ("wavefront", depth, threads), p
    _same(nx, ny, prec, (depth, 7, 2 * depth + 5, 11, 3), shape,
          rates=RATES if kind == "rates" else None, sr=kind == "stochastic",
          inplace=kind == "in place")


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,depth,rows", [(40, 30, 8, 7), (48, 9, 8, 16), (60, 12, 2, 5), (33, 70, 5, 64)])
def test_chosen_wavefront_on_narrow_lattices(prec, nx, ny, depth, rows):
    """A chosen depth and segment height on lattices no wider than one wave."""
    def shape(s):
        s.set_time_blocking(depth)
        s.set_fused_kernel("wavefront", rows)
        assert s.plain_launch()["steps_per_launch"] == depth
    _same(nx, ny, prec, (depth, 2 * depth + 1, 3), shape)


# the smallest lattices of the default rule (150000, 327680, 2^20 sites, 2^21 with
# stochastic rounding), whose short remainders and checks run through the tile
# kernel, and larger ones, whose do not
@pytest.mark.parametrize("prec,nx,ny,sr", [("fp64", 5000, 31, False), ("fp64", 450, 449, False),
                                           ("fp64", 570, 570, False), ("fp32", 600, 548, False),
                                           ("fp32", 701, 700, False), ("fp32", 850, 849, False),
                                           ("fp16", 1024, 1025, False), ("fp16", 1500, 1400, True)])
def test_short_calls_at_the_default_rule(prec, nx, ny, sr):
    """Calls of 2..11 steps, and checked calls of 2..21: states equal single
    steps', residuals up to the order of their sums (2^-53 per addition)."""
    from paper_2208_14870_amd import lbm
    _same(nx, ny, prec, tuple(range(2, 12)), None, (8 if prec == "fp16" else 12, 1), sr=sr)
    mat = P.Material.from_shear_poisson(0.9, 0.3)
    rng = np.random.default_rng(5)
    f0 = dev(rng.standard_normal((8, ny, nx)))
    g = rng.standard_normal((2, ny, nx)) * 1e-2
    g = [dev(a - a.mean()) for a in g]
    res = []
    for single in (False, True):
        s = lbm.Solver(nx, ny, prec)
        s.set_material(mat.lame_lambda, mat.lame_mu)
        if sr:
            s.set_stochastic_rounding(True, 7)
        s.set_body_force(*g)
        s.set_populations(f0)
        if single:
            s.set_time_blocking(1)
        r = [s.step_checked(n) for n in range(2, 22)]
        res.append((r, host(s.populations())))
        s.close()
    np.testing.assert_array_equal(res[0][1], res[1][1])
    np.testing.assert_allclose(res[0][0], res[1][0], rtol=nx * ny * 2.0 ** -52, atol=0)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny", [(100, 100), (31, 57), (3, 5)])
def test_general_rates_at_a_chosen_depth_on_small_lattices(prec, nx, ny):
    """Free rates have no tile kernel: a chosen depth runs through the
    small-lattice kernel where its tiles are no more than the compute units."""
    for depth in range(2, 9):
        def shape(s):
            s.set_time_blocking(depth)
            p = s.plain_launch()
            assert (p["kernel"], p["steps_per_launch"]) == ("square", depth), p
        _same(nx, ny, prec, (depth, 2 * depth + depth // 2, 3), shape, rates=RATES)


@pytest.mark.parametrize("prec,nx,ny,rates", [
    ("fp64", 200000, 1, None), ("fp32", 400001, 1, None), ("fp64", 7, 30000, RATES),
    ("fp32", 5, 40000, RATES), ("fp64", 60000, 3, RATES), ("fp16", 19, 20000, RATES)])
def test_thin_lattices_run_single_steps(prec, nx, ny, rates):
    """One row, and with free rates few columns or rows: one step per launch by
    default, checks included, in every length of call."""
    from paper_2208_14870_amd import lbm

    def shape(s):
        assert s.plain_launch()["kernel"] == "single", s.plain_launch()
    _same(nx, ny, prec, (1, 2, 5, 70), shape, rates=rates)
    s = lbm.Solver(nx, ny, prec)
    s.set_material(0.4, 0.3)
    g = dev(np.random.default_rng(1).standard_normal((ny, nx)) * 1e-3)
    s.set_body_force(g, g)
    r = []
    for one in (False, True):
        s.reset()
        if one:
            s.set_time_blocking(1)
        r.append([s.step_checked(n) for n in (2, 9, 70)] + [s.solve_to_tol(0.0, 20, 7)[1]])
    np.testing.assert_allclose(r[0], r[1], rtol=nx * ny * 2.0 ** -52, atol=0)
    s.close()


def test_half_storage_stays_with_tiles_that_cost_less():
    """A 64-column FP16 lattice of 2^24 sites and more, whose nominal kernel is the
    wavefront: its tiles cost less, and run it; states equal single steps."""
    from paper_2208_14870_amd import lbm
    import torch
    need_gpu()
    nx, ny = 64, 262200
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    f = torch.randn(2, ny, nx, generator=g, device="cuda", dtype=torch.float64) * 1e-4
    f -= f.mean(dim=(1, 2), keepdim=True)
    out = []
    for one in (False, True):
        s = lbm.Solver(nx, ny, "fp16")
        s.set_material(0.4, 0.3)
        s.set_body_force(f[0].contiguous(), f[1].contiguous())
        p = s.plain_launch()
        assert s.launch_config()["kernel"] == "wavefront"
        assert (p["kernel"], p["steps_per_launch"]) == ("tile", 8), p
        if one:
            s.set_time_blocking(1)
        for n in (8, 3, 13):
            s.step(n)
        r = s.step_checked(10)
        out.append((r, s.displacement()))
        s.close()
        del s
    for a, b in zip(out[0][1], out[1][1]):
        assert torch.equal(a, b)
    assert out[0][0] == pytest.approx(out[1][0], rel=nx * ny * 2.0 ** -52)
