"""The wavefront over the waves of a workgroup (k_wave): the depths, strips and
options that the library chooses by itself, against single steps bit for bit
(every level is rounded as a store would round it, so no tolerance)."""
import numpy as np
import pytest

from gpu_common import dev, host, need_gpu, say
from paper_2208_14870_amd import problem as P

pytestmark = pytest.mark.gpu


def _pair(nx, ny, prec, rates=None, steps=(), sr=False):
    """Populations after each of `steps` (cumulative): library default, and one
    step per launch."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    mat = P.Material.from_shear_poisson(0.9, 0.3)
    rng = np.random.default_rng(nx * 31 + ny)
    f0 = rng.standard_normal((8, ny, nx))
    g = rng.standard_normal((2, ny, nx)) * 1e-2
    g -= g.mean(axis=(1, 2), keepdims=True)
    out = []
    for single in (False, True):
        s = lbm.Solver(nx, ny, prec)
        if rates:
            s.set_rates(*rates)
        s.set_material(mat.lame_lambda, mat.lame_mu)
        if sr:
            s.set_stochastic_rounding(True, 7)
        s.set_body_force(dev(g[0]), dev(g[1]))
        s.set_populations(dev(f0))
        if single:
            s.set_time_blocking(1)
        res = []
        for n in steps:
            s.step(n)
            res.append(host(s.populations()))
        r = s.step_checked(13)
        res.append(host(s.populations()))
        s.close()
        out.append((res, r))
    for a, b in zip(out[0][0], out[1][0]):
        np.testing.assert_array_equal(a, b)
    # FP64 sums of the same values in another order: 2^-53 per addition, and a
    # square root
    assert out[0][1] == pytest.approx(out[1][1], rel=nx * ny * 2.0 ** -52)


# widths and heights below one strip, at and one beyond a strip's output
# columns (98 at twelve steps, 104 with two columns per lane, 108 for half
# storage at eight), odd and even
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 2), (20, 20), (97, 31), (98, 40), (99, 5), (104, 33),
                                   (105, 64), (108, 7), (109, 50), (250, 13)])
def test_general_rates_blocked_equal_single_steps(prec, nx, ny):
    """Free relaxation rates run through the wavefront by default: sequences
    whose remainders take every shallower depth."""
    say(f"general rates {prec} {nx}x{ny}")
    _pair(nx, ny, prec, rates=(0.3, 0.93, 0.9, 1.12), steps=(12, 9, 11, 2, 3, 5, 7, 8, 1, 23))


# the smallest lattices of the default rule, widths at a strip's edges
@pytest.mark.parametrize("prec,nx,ny", [("fp64", 980, 480), ("fp64", 981, 479), ("fp32", 1078, 1030),
                                        ("fp32", 1079, 1000), ("fp16", 4104, 4096)])
def test_default_depth_equals_single_steps(prec, nx, ny):
    """Twelve steps per launch (half storage eight) and the remainders 9..11,
    which take two launches."""
    say(f"default depth {prec} {nx}x{ny}")
    _pair(nx, ny, prec, steps=(12, 21, 10) if prec != "fp16" else (8, 11))


def test_default_depth_two_columns_per_lane():
    """A large FP32 lattice on an even width: two columns per lane."""
    say("default depth fp32 5826x5780")
    _pair(5826, 5780, "fp32", steps=(12, 5))


@pytest.mark.parametrize("nx,ny", [(4000, 3000), (4002, 2998)])
def test_default_depth_columns_per_lane_at_the_line(nx, ny):
    """FP32 at 12 M sites (two columns per lane) and just below (one), a full
    launch and remainders of one and two launches."""
    say(f"default depth fp32 {nx}x{ny}")
    _pair(nx, ny, "fp32", steps=(12, 5, 10))


def test_default_depth_stochastic_rounding():
    """Half storage with stochastic rounding at the default's eight steps."""
    say("default depth fp16 sr 4097x4096")
    _pair(4097, 4096, "fp16", steps=(8, 3), sr=True)


# one tile, one and two beyond a tile of 10 (twelve steps), 18 (eight) and 26
# (four) a side, more rows or columns than the other way round, and the largest
# square lattice of the small-lattice rule
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny", [(1, 3), (10, 10), (11, 31), (33, 9), (160, 161), (289, 288),
                                   (18, 3000), (2700, 20), (416, 416), (417, 416)])
def test_small_lattices_equal_single_steps(prec, nx, ny):
    """Default launches of small lattices at every depth the rule picks (deeper
    for fewer tiles), with every remainder."""
    say(f"small lattice {prec} {nx}x{ny}")
    _pair(nx, ny, prec, steps=(12, 11, 10, 9, 8, 7, 6, 5, 4, 3, 2, 1, 29))


def test_small_lattice_stochastic_rounding():
    say("small lattice fp16 sr 200x190")
    _pair(200, 190, "fp16", steps=(9, 13, 2), sr=True)
