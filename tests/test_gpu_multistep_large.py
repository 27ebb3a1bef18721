"""Runs advanced several steps per launch against single steps, bit for bit,
on grids where every storage's march is taken (binary16 and the double
states of more fields march on large grids only), and for combinations of
collision, fields, lattice and history beside each other."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_05668_amd import lbm  # noqa: E402
from test_gpu_multistep import SYSTEMS, initial, make, populations  # noqa: E402


def _same(a, b, counts):
    for n in counts:
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(populations(a), populations(b)), n


# ragged strips and segments; segments of few rows
@pytest.mark.parametrize("shape", [(1500, 1531), (61, 43397)])
@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "f16ne"])
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q5"])
@pytest.mark.parametrize("system", sorted(SYSTEMS))
def test_large_grids_of_every_state(system, lattice, storage, shape):
    if storage == "f16ne" and system == "gen_euler2d":
        pytest.skip("no such storage for the compiled systems")
    a, b = make(system, lattice, storage, shape), make(system, lattice, storage, shape)
    Q = initial(system, shape)
    for s in (a, b):
        s.init(Q)
    _same(a, b, (2, 3, 4, 11))


# the largest state that the deviations' march takes
@pytest.mark.parametrize("shape", [(700, 700), (1500, 1531), (61, 43397)])
def test_deviations_of_twelve_fields(shape):
    dx, dt, tau = lbm.recipe(64, "acoustic", 0.05, 5.0)
    a, b = (lbm.Stepper("cnsf_trk2d", "D2Q5", shape, tau, dt, dx, "f16ne", {"g_tau": 6.0, "mu": 0.001, "kappa": 0.001})
            for _ in range(2))
    Q = a.reference[:a.K][:, None, None] + 0.003 * np.random.default_rng(3).standard_normal((a.K,) + shape)
    for s in (a, b):
        s.init(Q)
    _same(a, b, (2, 3, 6, 7))
    assert torch.isfinite(a.moments()).all()


# two relaxation times read fields where some are attached, and elsewhere load
# words that nobody uses: flat grids march, of one row too
@pytest.mark.parametrize("fields", [(), ("grad_zb",), ("source",), ("grad_zb", "source")])
@pytest.mark.parametrize("storage,shape", [("f32", (101, 150)), ("f32", (397, 411)), ("f32", (3, 43400)), ("f32", (1, 200000)),
                                           ("f64", (700, 700)), ("f16", (1500, 1531))])
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q5"])
def test_two_relaxation_times_beside_fields(lattice, storage, shape, fields):
    a, b = (make("swe2d", lattice, storage, shape, trt_lambda=3.0 / 16.0) for _ in range(2))
    rng = np.random.default_rng(5)
    values = {"grad_zb": 0.01 * rng.standard_normal((2,) + shape), "source": 0.01 * rng.standard_normal((3,) + shape)}
    for s in (a, b):
        for name in fields:
            s.set_field(name, values[name])
        s.init(initial("swe2d", shape))
    _same(a, b, (4, 7))


@pytest.mark.parametrize("storage,shape", [("f32", (101, 150)), ("f32", (397, 411)), ("f32", (3, 43400)), ("f64", (700, 700)),
                                           ("f64", (1500, 1531)), ("f16", (1500, 1531))])
@pytest.mark.parametrize("system", ["swe2d", "euler2d", "neohooke2d"])
def test_fields_and_history_on_five_velocities(system, storage, shape):
    a, b = make(system, "D2Q5", storage, shape), make(system, "D2Q5", storage, shape)
    rng = np.random.default_rng(5)
    src = 0.01 * rng.standard_normal((a.K,) + shape)
    top = 0.01 * rng.standard_normal((2,) + shape)
    for s in (a, b):
        if system == "swe2d":
            s.set_field("grad_zb", top)
        s.set_field("source", src)
        s.init(initial(system, shape))
    _same(a, b, (5,))
    ha = torch.full((7, a.K) + shape, float("nan"), dtype=a.real, device="cuda")
    hb = torch.empty_like(ha)
    a.step_record(7, ha)
    for j in range(7):
        b.step_record(1, hb[j])
    assert torch.equal(ha, hb)
    assert torch.equal(populations(a), populations(b))
