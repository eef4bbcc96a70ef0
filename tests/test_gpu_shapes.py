"""Launch shapes that the library picks: what a solver runs by itself, what a
query says of it, and the way back to it."""
import numpy as np
import pytest

from paper_2208_14870_amd import problem as P
from gpu_common import dev, host, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
def test_reset_after_the_polish_switch_runs_the_narrow_shape(prec):
    """lbm_reset after a switch to FP64 is the solver as created: its launch
    shape and 25 steps from rest are those of a fresh solver, bit for bit (a
    size that steps through the tile kernel by default)."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    say(f"reset after polish {prec} 500x450")
    c = P.single_1024(0.3, 1, 1, n=450)
    gx, gy = (np.ascontiguousarray(np.pad(g, ((0, 0), (0, 50)))) for g in (c.gx, c.gy))
    gx, gy = P.remove_mean(gx), P.remove_mean(gy)

    def solver():
        s = lbm.Solver(500, 450, prec, with_polish=True)
        s.set_material(c.material.lame_lambda, c.material.lame_mu)
        s.set_body_force(dev(gx), dev(gy))
        return s

    a, b = solver(), solver()
    want = a.launch_config()
    a.set_polish(1e30)  # the switch at the first check
    a.solve_to_tol(0.0, 60, 20)
    assert a.current_precision == 0
    a.reset()
    assert a.launch_config() == want
    for s in (a, b):
        s.step(25)
    np.testing.assert_array_equal(host(a.populations()), host(b.populations()))
    a.close()
    b.close()


# what the default rule picks: sizes on both sides of its lines
@pytest.mark.parametrize("prec,nx,ny,want", [
    ("fp64", 64, 64, ("square", 12)), ("fp64", 400, 400, ("square", 4)),
    ("fp64", 420, 400, ("wavefront", 12)), ("fp32", 450, 450, ("tile", 8)),
    ("fp32", 600, 600, ("wavefront", 12)), ("fp16", 700, 700, ("tile", 8)),
    ("fp16", 1100, 1100, ("wavefront", 8)), ("fp32", 1024, 1024, ("wavefront", 12))])
def test_plain_launch_says_what_runs(prec, nx, ny, want):
    """The query names the kernel and depth of plain steps while nothing is
    chosen, and a chosen depth once there is one; the nominal shape is another
    question (lbm_get_launch_config)."""
    from paper_2208_14870_amd import lbm
    need_gpu()
    s = lbm.Solver(nx, ny, prec)
    got = s.plain_launch()
    assert (got["kernel"], got["steps_per_launch"]) == want
    if got["kernel"] == "square":
        assert got["rows"] == 32 - 2 * (want[1] - 1) and got["threads"] == 1024
        assert -(-nx // got["rows"]) * -(-ny // got["rows"]) <= 256
    s.set_time_blocking(3)
    assert s.plain_launch()["steps_per_launch"] == 3
    s.set_time_blocking(1)
    assert s.plain_launch()["kernel"] == "single" and s.plain_launch()["steps_per_launch"] == 1
    s.close()
