"""Initialisation, moments and reductions of the binary16 deviations by tiles
and by runs of cells: a narrow grid (runs) and the same fields repeated to a
wide one (tiles, on D2Q9) hold the same cells."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_05668_amd import lbm  # noqa: E402

SYSTEMS = {
    "swe2d": ({"g": 1.0}, [1, 0, 0]),
    "burgers2d": ({}, [0]),
    "neohooke2d": ({"rho0": 1.0, "mu_s": 1.0, "lambda_s": 2.0}, [1, 0, 0, 1, 0, 0]),
    "nse_trk2d": ({"cs_phys": 1.0, "mu": 0.01, "g_tau": 6.0}, [1] + [0] * 6),
}


def _stepper(system, lattice, shape):
    dx = 1.0 / 64
    return lbm.Stepper(system, lattice, shape, 0.5 + 0.2 * dx, 0.1 * dx, dx, "f16ne", SYSTEMS[system][0])


# widths one, ragged, one short of and one past a tile; times 64 all fill tiles
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q5"])
@pytest.mark.parametrize("system", sorted(SYSTEMS))
@pytest.mark.parametrize("nx", [1, 3, 20, 33])
def test_narrow_grids_hold_the_cells_of_wide_ones(system, lattice, nx):
    q0 = np.array(SYSTEMS[system][1], dtype=float)
    ny, repeat = 12, 64
    Q = q0[:, None, None] + 0.01 * np.random.default_rng(9).standard_normal((len(q0), ny, nx))
    wide = np.tile(Q, (1, 1, repeat))
    a, b = _stepper(system, lattice, (ny, nx)), _stepper(system, lattice, (ny, nx * repeat))
    a.init(Q)
    b.init(wide)
    for steps in (0, 3):
        a.step(steps)
        b.step(steps)
        ma, mb = a.moments(), b.moments()
        assert torch.isfinite(ma).all()
        assert torch.equal(ma.repeat(1, 1, repeat), mb)
        assert a.moments(dtype=torch.float32).repeat(1, 1, repeat).equal(b.moments(dtype=torch.float32))
        assert np.array_equal(a.reduce(lbm.RED_MAXSPEED), b.reduce(lbm.RED_MAXSPEED))
        assert np.array_equal(a.reduce(lbm.RED_RELLINF, Q), b.reduce(lbm.RED_RELLINF, wide))
        np.testing.assert_allclose(a.reduce(lbm.RED_RELL2, Q), b.reduce(lbm.RED_RELL2, wide), rtol=1e-12)
        np.testing.assert_allclose(repeat * a.reduce(lbm.RED_SUMS), b.reduce(lbm.RED_SUMS), rtol=1e-12, atol=1e-9)
        assert a.reduce(lbm.RED_NONFINITE)[0] == 0 and b.reduce(lbm.RED_NONFINITE)[0] == 0


def test_moments_of_a_grid_of_more_tiles_than_a_launch_holds():
    """One cell wide, 2^24 + 16 tiles high: each deviation is within 2^-11 of
    its value, at most twice the largest field, and five are summed."""
    ny = (1 << 26) + 64
    s = _stepper("burgers2d", "D2Q5", (ny, 1))
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    Q = 0.01 * torch.randn((1, ny, 1), device="cuda", dtype=torch.float64, generator=g)
    s.init(Q)
    assert (s.moments() - Q).abs().max() <= 5 * 2 * 2.0 ** -11 * Q.abs().max()
