"""Single-precision runs of states far from 1, up to the ends of the float
range.  A power-of-two change of units changes no mantissa, so the run in the
other units is the same run scaled; each of the 20 steps rounds every
population once (2^-24 of its size), and the two runs may round apart only
where a reciprocal or root differs in its last places."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_05668_amd import lbm  # noqa: E402

STEPS = 20


def _run(system, lattice, q0, unit, params):
    dx = 1.0 / 64
    q0 = np.array(q0) * unit
    s = lbm.Stepper(system, lattice, (40, 60), 0.5 + 0.4 * dx, 0.2 * dx, dx, "f32", params, reference=q0)
    noise = np.random.default_rng(11).standard_normal((len(q0), 40, 60))
    s.init(q0[:, None, None] + 0.01 * unit * noise)
    s.step(STEPS)
    return s.moments(absolute=False) / unit


# energy density and momenta: squares of them leave the float range
@pytest.mark.parametrize("unit", [2.0 ** -66, 2.0 ** -40, 2.0 ** 40, 2.0 ** 66])
def test_relativistic_fluid_in_other_units(unit):
    a = _run("relhydro2d", "D2Q9", [3.0, 1.2, 1.2], unit, {})
    b = _run("relhydro2d", "D2Q9", [3.0, 1.2, 1.2], 1.0, {})
    assert torch.isfinite(a).all()
    for k in range(3):
        assert (a[k] - b[k]).abs().max() <= STEPS * 2.0 ** -24 * b[k].abs().max()


# depth h and gravity 1 / h: the reciprocal of the depth is no normal float
@pytest.mark.parametrize("unit", [2.0 ** -100, 2.0 ** 100, 2.0 ** 126])
def test_shallow_water_in_other_units(unit):
    a = _run("swe2d", "D2Q9", [1.0, 0.0, 0.0], unit, {"g": 1.0 / unit})
    b = _run("swe2d", "D2Q9", [1.0, 0.0, 0.0], 1.0, {"g": 1.0})
    assert torch.isfinite(a).all()
    for k in range(3):
        assert (a[k] - b[k]).abs().max() <= STEPS * 2.0 ** -24 * b[k].abs().max()
