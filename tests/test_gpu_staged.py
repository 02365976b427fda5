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
