"""Mass and momentum over long runs. A periodic lattice conserves both (the
source term sums to zero over the sites), so the totals may drift only by
roundings that differ from site to site and step to step. A coefficient sum that
misses 1 by half a unit would act the same way at every step: n/2 units of the
total after n steps. The bounds are a quarter of that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402


def flow(nx, ny, seed):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:ny, 0:nx]
    rho = 1 + 1e-3 * np.sin(2 * np.pi * x / nx) + 1e-4 * rng.uniform(-1, 1, (ny, nx))
    return rho, 0.03 + 0.01 * np.sin(2 * np.pi * y / ny), -0.02 + 0.005 * np.cos(2 * np.pi * x / nx)


@pytest.mark.parametrize("dtype", ["f32", "f32s"])
@pytest.mark.parametrize("model", [lbm.MODEL_FORCING, lbm.MODEL_EQUILIBRIUM])
@pytest.mark.parametrize("tau", [0.552, 0.6335, 0.9, 1.31, 1.4881])
def test_momentum_after_1000_steps(dtype, model, tau):
    steps, unit = 1000, 2.0 ** -24
    with lbm.Lattice(70, 58, tau, 0.25, dtype, model=model) as L:
        L.init(*flow(70, 58, 1))
        before = L.totals()
        after = L.step(steps).totals()
    for k in (1, 2):
        assert abs(after[k] / before[k] - 1) <= steps * unit / 8, (dtype, model, tau, k, after[k] / before[k] - 1)


@pytest.mark.parametrize("tau,c2", [(0.55, 0.1), (0.7, 0.1), (0.7, 0.55)])
def test_mass_of_the_equilibrium_model_fp64(tau, c2):
    steps, unit = 2000, 2.0 ** -53
    with lbm.Lattice(70, 58, tau, c2, "f64", model=lbm.MODEL_EQUILIBRIUM) as L:
        L.init(*flow(70, 58, 2))
        before = L.totals()
        after = L.step(steps).totals()
    assert abs(after[0] / before[0] - 1) <= steps * unit / 8, (tau, c2, after[0] / before[0] - 1)
