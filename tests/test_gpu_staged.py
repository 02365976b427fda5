"""The passes on in-place staged transforms against the FP64 oracle, at the
lengths where their stages, tiles and rules can go wrong.

Tolerance: a run of k steps chains 14 k float32 transforms of a few thousand
points, each about 1e-7 log2(n) relative, added at random: 1e-7 * 12 *
sqrt(14 * 4) is 9e-6 at 4 steps; 2e-5 leaves a factor two."""
import numpy as np
import pytest

from oracle import Oracle
from oracle.adjoint import AdjointOracle
from paper_1408_4675_amd import scenarios as sc
from tests._parity import compare_outputs

pytestmark = pytest.mark.gpu

TOL = 2e-5
STEPS = 4


@pytest.fixture(scope="module")
def kw():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1408_4675_amd import _abi as A
    from paper_1408_4675_amd.simulation import Simulation
    A.load()
    return A, Simulation


def _check(kw, scen, **sim_args):
    A, Simulation = kw
    print("\n[case] %s" % scen.name, flush=True)
    sim = Simulation(scen, **sim_args)
    sim.step(STEPS)
    orc = Oracle(scen)
    orc.step(STEPS)
    errs, _ = compare_outputs(sim, orc, scen, [])
    sim.close()
    for k, e in errs.items():
        assert e <= TOL, (k, e)


def _case(nx, ny, nz, medium, mask=False):
    return sc.small_case(nx, ny, nz, seed=nx + 7 * ny + 31 * nz, heterogeneous=medium == "maps",
                         nonlinear=medium != "lossless", absorbing=medium != "lossless", pml=1,
                         steps=STEPS, sensor_mask=mask)


# one stage's worth (the first of radix 1), every radix as the last stage, two
# and three stages, odd lengths (no Nyquist plane), and tiles wider than the grid
COLUMNS = [4, 5, 9, 12, 15, 16, 18, 27, 32, 50, 64, 75, 81, 100, 120, 125, 128, 135, 162, 180,
           225, 240, 243, 250, 256, 375, 486, 500, 600, 625, 900]


@pytest.mark.parametrize("n", COLUMNS)
@pytest.mark.parametrize("medium", ["maps", "water", "lossless"])
def test_z_columns(kw, n, medium):
    """The fused z pass in every mode of a step: gradient (three outputs a
    block, or one), divergence, absorption apart (maps) and merged (water)."""
    _check(kw, _case(8 if n > 64 else 40, 6, n, medium))


@pytest.mark.parametrize("n", COLUMNS)
def test_y_columns(kw, n):
    """The y pass, its packed column 0 included (kx = 0 and Nyquist)."""
    _check(kw, _case(8 if n > 64 else 36, n, 5, "maps"))


def test_kappa_beyond_the_polynomial(kw):
    """Time steps whose kappa argument leaves the polynomial's range keep the
    pass that evaluates the sine."""
    scen = _case(12, 10, 18, "lossless")
    g = sc.Grid(12, 10, 18, 1e-4, 1e-4, 1e-4, dt=0.0, cfl=0.75, pml_size=(0, 0, 0))
    _check(kw, scen.replace(grid=g))


@pytest.mark.parametrize("shape", [(16, 45, 75), (18, 8, 128), (24, 100, 9)])
def test_reverse_step(kw, shape):
    """The transposed operators on staged z and y passes."""
    from paper_1408_4675_amd.adjoint import focus_gradient
    T = 8
    scen = sc.small_case(*shape, seed=3, pml=2, steps=T, amp=2.0e6, n_elements=3)
    scen = scen.replace(sensor=sc.Sensor(record=sc.REC_INTENSITY, record_start=3))
    w = np.random.default_rng(5).standard_normal(scen.grid.npts)
    ref = AdjointOracle(scen, w, workers=4)
    ref.forward()
    gr = ref.backward()
    out = focus_gradient(scen, w, checkpoint_every=3)
    e = np.linalg.norm(out["source_gradient"] - gr["dJds"]) / np.linalg.norm(gr["dJds"])
    print("[case] %s dJ/ds %.2e" % (scen.name, e), flush=True)
    assert e <= TOL


# rows of a generic length (two and three stages, one, a remainder of rows), the velocity
# pass on planes or, with few large ones, on rows; and planes alone
@pytest.mark.parametrize("shape", [(250, 20, 10), (250, 36, 6), (810, 6, 8), (90, 48, 15), (128, 36, 8), (64, 12, 9)])
@pytest.mark.parametrize("absorbing", [True, False])
def test_reverse_x_passes(kw, shape, absorbing):
    """The reverse x passes on staged rows and planes, with and without absorption."""
    from paper_1408_4675_amd.adjoint import focus_gradient
    scen = sc.small_case(*shape, seed=4, pml=2, steps=6, amp=2.0e6, n_elements=3, absorbing=absorbing)
    scen = scen.replace(sensor=sc.Sensor(record=sc.REC_INTENSITY, record_start=3))
    w = np.random.default_rng(6).standard_normal(scen.grid.npts)
    ref = AdjointOracle(scen, w, workers=4)
    ref.forward()
    gr = ref.backward()
    out = focus_gradient(scen, w, checkpoint_every=3)
    e = np.linalg.norm(out["source_gradient"] - gr["dJds"]) / np.linalg.norm(gr["dJds"])
    print("[case] %s dJ/ds %.2e" % (scen.name, e), flush=True)
    assert e <= TOL


def _smooth(n):
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            return n
        n += 1


# packed row lengths nx / 2: one stage (the update's of radix 1), two, three, every
# radix of the last stage, odd ones (no partner of its own in the middle)
ROWS = [2, 3, 4, 5, 8, 9, 12, 15, 16, 18, 24, 25, 32, 45, 60, 64, 75, 81, 90, 96, 100, 125, 128, 135, 200,
        225, 243, 250, 405, 500]


@pytest.mark.parametrize("m", ROWS)
@pytest.mark.parametrize("medium", ["maps", "water", "lossless"])
def test_x_rows_on_planes(kw, m, medium):
    """x passes on z planes (the velocity's, on small planes all three), with mass
    source points and every point recorded."""
    _check(kw, _case(2 * m, 6 if m < 200 else 5, 5, medium))


@pytest.mark.parametrize("m", [15, 25, 45, 75, 80, 90, 100, 125, 135, 200, 225, 250, 405, 500])
@pytest.mark.parametrize("medium", ["maps", "water", "lossless"])
@pytest.mark.parametrize("mask", [False, True])
def test_x_rows(kw, m, medium, mask):
    """x passes on rows (planes too large for few blocks): full and ragged blocks,
    mass source points, every point recorded or a mask with its series."""
    _check(kw, _case(2 * m, _smooth(4097 // m + 1), 4, medium, mask))


@pytest.mark.parametrize("shape", [(64, 64, 48), (96, 96, 50), (50, 45, 50), (128, 128, 48)])
def test_velocity_on_large_planes(kw, shape):
    """Velocity planes of the usual sizes (blocks of 512 and 1024 threads)."""
    _check(kw, _case(*shape, "maps"))


@pytest.mark.parametrize("shape", [(30, 8, 6), (100, 90, 4)], ids=["planes", "rows"])
@pytest.mark.parametrize("kind,axis", [(sc.SOURCE_FORCE, 0), (sc.SOURCE_FORCE, 2), (sc.SOURCE_PRESSURE, 0)])
@pytest.mark.parametrize("medium", ["maps", "water", "lossless"])
def test_sources_and_sensors_between_the_transforms(kw, shape, kind, axis, medium):
    """Force and pressure sources, and mask sensors with velocity series, harmonics and
    p_min: written and read between the inverse and the forward x transform."""
    import dataclasses
    scen = _case(*shape, medium, mask=True)
    rec = (sc.REC_P_MAX | sc.REC_P_MIN | sc.REC_P_RMS | sc.REC_P_SERIES | sc.REC_U_SERIES |
           sc.REC_HARMONICS | sc.REC_P_FINAL | sc.REC_U_FINAL)
    sen = dataclasses.replace(scen.sensor, record=rec, series_capacity=STEPS, n_harmonics=2)
    # (a force of 1e6 m/s^2 gives dt F of about 0.02 m/s)
    src = dataclasses.replace(scen.source, kind=kind, axis=axis)
    _check(kw, scen.replace(source=src, sensor=sen))


@pytest.mark.parametrize("shape", [(30, 8, 6), (100, 90, 4), (64, 64, 48)])
def test_forced_schedules_agree(kw, shape):
    """The engines, forced with kw_set_plan, and the staged passes give the same fields to
    rounding (TOL), and a tuned schedule given as a hint changes nothing there."""
    A, Simulation = kw
    scen = _case(*shape, "maps")
    outs = []
    for mode in ("staged", "hint", "engine"):
        sim = Simulation(scen, tune=False)
        if mode != "staged":
            call = sim.lib.kw_suggest_plan if mode == "hint" else sim.lib.kw_set_plan
            for axis, n in enumerate((shape[0] // 2, shape[1], shape[2])):
                rad = [2, n // 2] if n % 2 == 0 and n // 2 <= 16 else None
                if rad or mode == "engine":
                    sim._plan(call, axis, rad, 0)
        sim.step(STEPS)
        outs.append(sim.gather(A.KW_REC_P_FINAL, device=False).astype(np.float64))
        sim.close()
    if shape == (30, 8, 6):
        assert np.linalg.norm(outs[1] - outs[0]) <= TOL * np.linalg.norm(outs[0])
    assert np.linalg.norm(outs[2] - outs[0]) <= TOL * np.linalg.norm(outs[0])
