"""Runs advanced several steps per launch against the same runs advanced one
step per launch: every stored population and every recorded moment equal bit
for bit, for grids at the edges of the strips and segments (one column or row,
just below and above a strip's width, ragged tiles), each storage type, with
and without coefficient and source fields."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_05668_amd import inputs, lbm  # noqa: E402

SYSTEMS = {
    "swe2d": ("acoustic", 0.2, 2.0, None, {"g": 1.0}, [1, 0, 0]),
    "burgers2d": ("acoustic", 0.2, 2.0, None, {}, [0]),
    "euler2d": ("acoustic", 0.05, 5.0, None, {"gamma": 1.4}, [1, 3, 3, 1 / (1.4 * 0.4) + 9]),
    "maxwell2d": ("acoustic", 0.2, 0.2, None, {"c": 1.0}, [0, 0, 0]),
    "allencahn_trk2d": ("diffusive", 1.9, 50.0, 6.0, {"nu": 0.01, "R": 1.0}, [0, 0, 0]),
    "relhydro2d": ("acoustic", 0.2, 0.2, None, {}, [3, 1.2, 1.2]),
    "nse_trk2d": ("diffusive", 2.0, 90.0, 6.0, {"cs_phys": 1.0, "mu": 0.01}, [1] + [0] * 6),
    "advdiff_trk2d": ("diffusive", 1.9, 50.0, 6.0, {"ax": 0.1, "ay": 0.05, "nu": 0.01, "R": 0.3}, [1, 0, 0]),
    "neohooke2d": ("acoustic", 0.1, 20.0, None, {"rho0": 1.0, "mu_s": 1.0, "lambda_s": 2.0}, [1, 0, 0, 1, 0, 0]),
    "gen_euler2d": ("acoustic", 0.05, 5.0, None, {}, [1, 3, 3, 1 / (1.4 * 0.4) + 9]),
}
# up to 1024 squares of 12 x 12 cells the squares; else (thin grids, states too
# large for them) at most 700 strips' rows (62 columns each) two steps a launch,
# from 2000 on the most steps a launch, in between one
SHAPES = [(1, 1), (2, 3), (130, 1), (1, 130), (61, 59), (40, 60), (9, 62), (70, 64), (33, 121), (101, 150), (40, 1200),
          (2100, 30), (3, 43400), (210, 640), (67, 2011)]


def make(system, lattice, storage, shape, **more):
    scaling, f, tau_r, g_tau, params, _ = SYSTEMS[system]
    dx, dt, tau = lbm.recipe(64, scaling, f, tau_r)
    if g_tau is not None:
        params = dict(params, g_tau=g_tau)
    params = dict(params, **more)
    return lbm.Stepper(system, lattice, shape, tau, dt, dx, storage, params)


def initial(system, shape, seed=3):
    q0 = np.array(SYSTEMS[system][5], dtype=float)
    rng = np.random.default_rng(seed)
    return q0[:, None, None] + 0.01 * rng.standard_normal((len(q0),) + shape)


def populations(s):
    """The valid populations of the current buffer, [cells, K Q] (binary16
    deviations: and the moments)."""
    if s.storage == "f16ne":
        b = s.snapshot()
        n = s.K * s.Q * ((s.C + 63) // 64) * 64 * 2
        g = b[:n].view(torch.int16).reshape(-1, s.K * s.Q, 64).permute(0, 2, 1).reshape(-1, s.K * s.Q)[:s.C]
        m = b[(n + 255) // 256 * 256:].view(torch.int32).reshape(s.K, s.C)
        return torch.cat([g.flatten().int(), m.flatten()])
    el = {"f64": torch.int64, "f32": torch.int32, "f16": torch.int16}[s.storage]
    v = s.snapshot().view(el).reshape(-1, s.K * s.Q, 64).permute(0, 2, 1).reshape(-1, s.K * s.Q)
    return v[:s.C]


@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "f16ne"])
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q5"])
@pytest.mark.parametrize("system", sorted(SYSTEMS))
def test_several_steps_per_launch_are_bit_identical(system, lattice, storage):
    if storage == "f16ne" and system == "gen_euler2d":
        pytest.skip("no such storage for the compiled systems")
    for shape in SHAPES:
        print(system, lattice, storage, shape, flush=True)
        a, b = make(system, lattice, storage, shape), make(system, lattice, storage, shape)
        Q = initial(system, shape)
        for s in (a, b):
            s.init(Q)
        for n in (2, 3, 4, 11):
            a.step(n)
            for _ in range(n):
                b.step(1)
            assert a.steps == b.steps
            assert torch.isfinite(a.moments()).all()
            assert torch.equal(populations(a), populations(b)), (shape, n)


@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("system", ["swe2d", "advdiff_trk2d", "neohooke2d"])
def test_fields_and_history_in_several_steps_per_launch(system, storage):
    for shape in [(1, 1), (2, 3), (61, 59), (33, 121), (101, 150), (3, 43400), (210, 640)]:
        print(system, storage, shape, flush=True)
        a, b = make(system, "D2Q9", storage, shape), make(system, "D2Q9", storage, shape)
        rng = np.random.default_rng(5)
        src = 0.01 * rng.standard_normal((a.K,) + shape)
        top = 0.01 * rng.standard_normal((2,) + shape)
        for s in (a, b):
            if system == "swe2d":
                s.set_field("grad_zb", top)
            s.set_field("source", src)
            s.init(initial(system, shape))
        a.step(5)
        for _ in range(5):
            b.step(1)
        assert torch.equal(populations(a), populations(b)), shape
        ha = torch.full((7, a.K) + shape, float("nan"), dtype=a.real, device="cuda")
        hb = torch.empty_like(ha)
        a.step_record(7, ha)
        for j in range(7):
            b.step_record(1, hb[j])
        assert torch.equal(ha, hb), shape
        assert torch.equal(populations(a), populations(b)), shape


def test_topography_in_several_steps_per_launch_of_binary16_deviations():
    for shape in [(3, 43400), (210, 640)]:
        print("swe2d f16ne", shape, flush=True)
        a, b = make("swe2d", "D2Q9", "f16ne", shape), make("swe2d", "D2Q9", "f16ne", shape)
        top = 0.01 * np.random.default_rng(5).standard_normal((2,) + shape)
        for s in (a, b):
            s.set_field("grad_zb", top)
            s.init(initial("swe2d", shape))
        a.step(7)
        for _ in range(7):
            b.step(1)
        assert torch.equal(populations(a), populations(b)), shape


@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("system,lattice", [("swe2d", "D2Q9"), ("euler2d", "D2Q5")])
def test_two_relaxation_times_in_several_steps_per_launch(system, lattice, storage):
    for shape in [(2, 3), (33, 121), (210, 640)]:
        print(system, lattice, storage, shape, flush=True)
        a, b = (make(system, lattice, storage, shape, trt_lambda=3.0 / 16.0) for _ in range(2))
        for s in (a, b):
            s.init(initial(system, shape))
        a.step(9)
        for _ in range(9):
            b.step(1)
        assert torch.equal(populations(a), populations(b)), shape


# squares of 16 x 16 cells store 8 x 8 of them after five steps, 10 x 10 after
# four, 12 x 12 after three: one square, a ragged second one, grids on both
# sides of the changes from five to four to three steps and to other kernels
@pytest.mark.parametrize("shape", [(8, 8), (9, 17), (128, 128), (129, 128), (160, 160), (192, 192), (200, 200),
                                   (384, 384), (384, 385)])
@pytest.mark.parametrize("system,lattice,storage", [("swe2d", "D2Q9", "f32"), ("advdiff_trk2d", "D2Q5", "f64"),
                                                    ("neohooke2d", "D2Q9", "f16"), ("nse_trk2d", "D2Q5", "f32")])
def test_small_grids_in_several_steps_per_launch(system, lattice, storage, shape):
    a, b = make(system, lattice, storage, shape), make(system, lattice, storage, shape)
    for s in (a, b):
        s.init(initial(system, shape))
    for n in (2, 4, 5, 13):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.isfinite(a.moments()).all()
        assert torch.equal(populations(a), populations(b)), n


# beyond 1024 squares of 12 x 12: the marching kernel, ragged strips and segments
@pytest.mark.parametrize("shape", [(397, 411), (1201, 130)])
@pytest.mark.parametrize("trt", [0.0, 3.0 / 16.0])
@pytest.mark.parametrize("system,lattice,storage", [("swe2d", "D2Q9", "f32"), ("euler2d", "D2Q5", "f64"),
                                                    ("neohooke2d", "D2Q9", "f16"), ("nse_trk2d", "D2Q5", "f32")])
def test_large_grids_in_several_steps_per_launch(system, lattice, storage, trt, shape):
    a, b = (make(system, lattice, storage, shape, trt_lambda=trt) for _ in range(2))
    for s in (a, b):
        s.init(initial(system, shape))
    for n in (2, 3, 4, 11):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(populations(a), populations(b)), n


@pytest.mark.parametrize("shape", [(397, 411), (1201, 130)])
@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
def test_fields_and_history_of_large_grids_in_several_steps_per_launch(storage, shape):
    a, b = make("swe2d", "D2Q9", storage, shape), make("swe2d", "D2Q9", storage, shape)
    rng = np.random.default_rng(5)
    src = 0.01 * rng.standard_normal((a.K,) + shape)
    top = 0.01 * rng.standard_normal((2,) + shape)
    for s in (a, b):
        s.set_field("grad_zb", top)
        s.set_field("source", src)
        s.init(initial("swe2d", shape))
    a.step(6)
    for _ in range(6):
        b.step(1)
    ha = torch.full((7, a.K) + shape, float("nan"), dtype=a.real, device="cuda")
    hb = torch.empty_like(ha)
    a.step_record(7, ha)
    for j in range(7):
        b.step_record(1, hb[j])
    assert torch.equal(ha, hb)
    assert torch.equal(populations(a), populations(b))
