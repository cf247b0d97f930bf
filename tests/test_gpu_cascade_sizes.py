"""Cascade passes at the widths where a strip's last columns, a lane's columns
and the boundary columns fall differently, and two-step passes between the
sizes of the other kernels, and pools: the bits of single steps (see cascade_sizes.py; the
passes that these sizes take are checked in test_routes.py)."""
import numpy as np
import pytest

import cascade_sizes
from paper_0707_2437_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402

SINGLE = (2, 8, 0, 16 | 2)  # single-step vertical stack


def run(nx, ny, dtype, calls, tile=None, model=None, field=False, inlet=None):
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    r = lambda a: a * torch.randn(ny, nx, generator=g, dtype=torch.float64, device="cuda")  # noqa: E731
    f = 1.0 + r(0.01), r(0.02), r(0.02)
    with lbm.Lattice(nx, ny, 0.7, 0.3, dtype) as L:
        if model is not None:
            L.set_model(model)
        if field:
            L.set_c2_field(workloads.lens_c2_field(nx, ny, 0.3, noise=0.05, seed=1))
        if inlet:
            L.set_x_boundaries(lbm.XBC_INLET_OUTLET, *inlet)
        if tile:
            L.set_tile(*tile)
        L.set_stream(torch.cuda.current_stream())
        L.init_device(*f)
        for n in calls:
            L.step(n)
        return L.get_f()


@pytest.mark.parametrize("dtype,steps,nx,ny", [(d, s, nx, ny) for (d, s), sizes in cascade_sizes.SIZES.items()
                                               for nx, ny in sizes])
def test_cascade_bits_at_strip_widths(dtype, steps, nx, ny):
    for d, s, x, y, name, kw in cascade_sizes.cases():
        if (d, s, x, y) == (dtype, steps, nx, ny):
            ref = run(nx, ny, dtype, (2 * steps + 5,), SINGLE, **kw)
            assert np.array_equal(run(nx, ny, dtype, (steps, steps + 5), **kw), ref), (dtype, steps, nx, ny, name)


@pytest.mark.parametrize("dtype,nx,ny,kw", cascade_sizes.pair_cases())
def test_two_step_bits_between_block_and_cascade_sizes(dtype, nx, ny, kw):
    ref = run(nx, ny, dtype, (7,), SINGLE, **kw)
    assert np.array_equal(run(nx, ny, dtype, (7,), **kw), ref)
    assert np.array_equal(run(nx, ny, dtype, (2, 5), **kw), ref)


def alone(k, dtype, steps):
    nx, ny = cascade_sizes.POOL_SHAPES[k]
    with lbm.Lattice(nx, ny, 0.6 + 0.05 * k, 0.1 + 0.02 * k, dtype) as L:
        L.set_tile(*SINGLE)
        L.set_stream(torch.cuda.current_stream())
        L.init_device(*pool_fields(k))
        return L.step(steps).get_f()


def pool_fields(k):
    nx, ny = cascade_sizes.POOL_SHAPES[k]
    g = torch.Generator(device="cuda").manual_seed(k)
    r = lambda a: a * torch.randn(ny, nx, generator=g, dtype=torch.float64, device="cuda")  # noqa: E731
    return 1.0 + r(0.01), r(0.02), r(0.02)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s"])
@pytest.mark.parametrize("mode", [lbm.GROUPED, lbm.GRAPH, lbm.PERSISTENT])
def test_pool_cascade_bits(dtype, mode):
    shapes = cascade_sizes.POOL_SHAPES
    with lbm.Pool(sum(lbm.Pool.slot_bytes(nx, ny, dtype) for nx, ny in shapes), dtype) as P:
        P.set_mode(mode)
        slots = []
        for k, (nx, ny) in enumerate(shapes):
            slots.append(P.add(nx, ny, 0.6 + 0.05 * k, 0.1 + 0.02 * k))
            f = pool_fields(k)
            torch.cuda.synchronize()
            P.init_device(slots[-1], *f)
            P.sync()
        for counts in cascade_sizes.POOL_COUNTS:
            P.step(slots, np.array(counts, dtype=np.int32))
        for k, s in enumerate(slots):
            assert P.time(s) == sum(c[k] for c in cascade_sizes.POOL_COUNTS)
            assert np.array_equal(P.get_f(s), alone(k, dtype, P.time(s))), (dtype, mode, shapes[k])
