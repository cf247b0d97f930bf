"""The cascade kernel (four or eight steps of Eq. 5 per pass, rows falling
through the levels that four waves hold in registers), which the default shape
takes on large lattices, gives the bits of single steps: strips one column
short of, at and past a strip's width (112 or 240 columns, 96 with eight steps), lattices narrower than a strip (whose lanes
wrap several times), lower than a pass's halo (whose rows wrap several times)
and with ragged last chunks; every stored type, the altered-equilibrium model,
c2 fields; step counts with every remainder of four."""
import numpy as np
import pytest

from paper_0707_2437_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402

SINGLE = (2, 8, 0, 16 | 2)  # single-step vertical stack


def fields(nx, ny, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda a: a * torch.randn(ny, nx, generator=g, dtype=torch.float64, device="cuda")  # noqa: E731
    return 1.0 + r(0.01), r(0.02), r(0.02)


def run(nx, ny, dtype, calls, f, tile=None, model=None, c2_field=None, inlet=None):
    with lbm.Lattice(nx, ny, 0.7, 0.3, dtype) as L:
        if model is not None:
            L.set_model(model)
        if c2_field is not None:
            L.set_c2_field(c2_field)
        if inlet:
            L.set_x_boundaries(lbm.XBC_INLET_OUTLET, *inlet)
        if tile:
            L.set_tile(*tile)
        L.set_stream(torch.cuda.current_stream())
        L.init_device(*f)
        for n in calls:
            L.step(n)
        assert L.time == sum(calls)
        return L.get_f()


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx,ny", [(5, 260003), (49, 20011), (112, 10007), (113, 9001), (300001, 3), (260003, 4),
                                   (1103, 1021), (2353, 2251)])
def test_cascade_bitwise_equals_single_steps(dtype, nx, ny):
    f = fields(nx, ny, nx + ny)
    for calls in ((8,), (4, 5), (7, 6)):
        ref = run(nx, ny, dtype, (sum(calls),), f, SINGLE)
        got = run(nx, ny, dtype, calls, f)
        assert np.array_equal(got, ref), (dtype, nx, ny, calls)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx,ny", [(95, 52009), (96, 52003), (97, 52001), (193, 30011), (239, 30011), (241, 30013),
                                   (260003, 19), (4003, 1501)])
def test_cascade_eight_steps_and_remainders_bitwise(dtype, nx, ny):
    f = fields(nx, ny, nx + ny)
    ref = run(nx, ny, dtype, (29,), f, SINGLE)
    for calls in ((29,), (8, 12, 9)):  # 3 passes of eight, one of four, a single step
        got = run(nx, ny, dtype, calls, f)
        assert np.array_equal(got, ref), (dtype, nx, ny, calls)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx,ny", [(1103, 1021), (2353, 2251)])
def test_cascade_models_and_fields_bitwise(dtype, nx, ny):
    f = fields(nx, ny, 3)
    c2 = workloads.lens_c2_field(nx, ny, 0.3, noise=0.05, seed=1)
    for kw in ({"model": lbm.MODEL_EQUILIBRIUM}, {"c2_field": c2}):
        ref = run(nx, ny, dtype, (9,), f, SINGLE, **kw)
        got = run(nx, ny, dtype, (9,), f, **kw)
        assert np.array_equal(got, ref), (dtype, nx, ny, list(kw))


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx,ny", [(95, 60013), (97, 60013), (113, 60013), (241, 30013), (200003, 21), (2353, 2251)])
def test_cascade_inlet_bitwise(dtype, nx, ny):
    f = fields(nx, ny, nx)
    for kw in ({}, {"model": lbm.MODEL_EQUILIBRIUM}):
        ref = run(nx, ny, dtype, (3, 26), f, SINGLE, inlet=(0.02, 17.0), **kw)
        for calls in ((3, 26), (8, 4, 16, 1)):
            got = run(nx, ny, dtype, calls, f, inlet=(0.02, 17.0), **kw)
            assert np.array_equal(got, ref), (dtype, nx, ny, calls)
