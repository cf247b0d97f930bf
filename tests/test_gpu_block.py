"""The block kernel (many steps of Eq. 5 per launch on tiles of up to 16 rows
and 64 columns), which the default shape takes on small lattices, gives the
bits of single steps: lattices of at most 16 rows, held whole in y, and taller
ones with ragged last groups; widths around a strip's columns; every stored
type, both models, c2 fields, inlet/outlet boundaries; counts that leave
remainders, over several calls."""
import numpy as np
import pytest

from gpu_util import smooth_random_state
from paper_0707_2437_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402

SINGLE = (2, 8, 0, 16 | 2)  # single-step vertical stack
DTYPES = ["f64", "f32", "f32s", "f16s"]


def run(nx, ny, dtype, calls, tile=None, model=None, c2_field=None, inlet=None):
    with lbm.Lattice(nx, ny, 0.7, 0.3, dtype) as L:
        if model is not None:
            L.set_model(model)
        if c2_field is not None:
            L.set_c2_field(c2_field)
        if inlet is not None:
            L.set_x_boundaries(lbm.XBC_INLET_OUTLET, *inlet)
        if tile:
            L.set_tile(*tile)
        L.init(*smooth_random_state(nx, ny, seed=nx * 7 + ny))
        for n in calls:
            L.step(n)
        assert L.time == sum(calls)
        return L.get_f()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 4), (16, 4), (400, 4), (401, 5), (97, 15), (300, 16), (4000, 4), (40001, 3),
                                   (3, 17), (64, 64), (61, 18), (130, 77), (1000, 17), (250, 250)])
def test_block_bitwise_equals_single_steps(dtype, nx, ny):
    ref = run(nx, ny, dtype, (29,), SINGLE)
    for calls in ((29,), (2, 13, 1, 3, 10)):
        assert np.array_equal(run(nx, ny, dtype, calls), ref), (dtype, nx, ny, calls)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("nx,ny", [(5, 4), (403, 4), (97, 16), (64, 50), (333, 120)])
def test_block_options_bitwise(dtype, nx, ny):
    c2 = workloads.lens_c2_field(nx, ny, 0.3, noise=0.05, seed=1)
    for kw in ({"model": lbm.MODEL_EQUILIBRIUM}, {"c2_field": c2}, {"inlet": (0.01, 17.0)},
               {"inlet": (0.9, 9.0), "model": lbm.MODEL_EQUILIBRIUM}, {"inlet": (0.01, 17.0), "c2_field": c2}):
        ref = run(nx, ny, dtype, (23,), SINGLE, **kw)
        for calls in ((23,), (1, 9, 13)):
            assert np.array_equal(run(nx, ny, dtype, calls, **kw), ref), (dtype, nx, ny, calls, list(kw))
