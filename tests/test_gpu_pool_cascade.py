"""Pools whose default tile takes cascade passes (four steps of every listed
lattice per launch): every slot has the bits it gets alone in single steps, for
lattices of widths around a strip's columns, lower than a pass's halo and
taller than a chunk, with per-slot counts of every remainder of four (some
below one pass, some zero), over consecutive calls, in grouped, graph and persistent
launches, mixed with calls of two-step and single-step tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402

SHAPES = [(700, 500), (1001, 333), (49, 5003), (113, 3001), (5, 60003), (640, 641), (60001, 3), (112, 1700)]
COUNTS = [(8, 13, 6, 7, 3, 0, 21, 4), (5, 4, 11, 1, 10, 16, 2, 9), (8, 13, 6, 7, 3, 0, 21, 4)]
SINGLE = (2, 8, 0, 16 | 2)


def fields(nx, ny, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda a: a * torch.randn(ny, nx, generator=g, dtype=torch.float64, device="cuda")  # noqa: E731
    return 1.0 + r(0.01), r(0.02), r(0.02)


def alone(k, dtype, steps):
    nx, ny = SHAPES[k]
    with lbm.Lattice(nx, ny, 0.6 + 0.1 * k, 0.1 + 0.05 * k, dtype) as L:
        L.set_tile(*SINGLE)
        L.set_stream(torch.cuda.current_stream())
        L.init_device(*fields(nx, ny, k))
        return L.step(steps).get_f()


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s"])
@pytest.mark.parametrize("mode", [lbm.GROUPED, lbm.GRAPH, lbm.PERSISTENT])
def test_pool_cascade_bitwise(dtype, mode):
    total = sum(lbm.Pool.slot_bytes(nx, ny, dtype) for nx, ny in SHAPES)
    with lbm.Pool(total, dtype) as P:
        P.set_mode(mode)
        slots = []
        for k, (nx, ny) in enumerate(SHAPES):
            slots.append(P.add(nx, ny, 0.6 + 0.1 * k, 0.1 + 0.05 * k))
            f = fields(nx, ny, k)
            torch.cuda.synchronize()
            P.init_device(slots[-1], *f)
            P.sync()
        tile = P.get_tile()
        for call, counts in enumerate(COUNTS):
            if call == 1:  # the passes' buffer phases carry over other kinds of launches
                P.set_tile(2, 8, 2)
                P.step(slots, 3)
                P.set_tile(1, 12, 32 | 2)
                P.step(slots, 5)
                P.set_tile(*tile)
            P.step(slots, np.array(counts, dtype=np.int32))
        assert [P.time(s) for s in slots] == [sum(c[k] for c in COUNTS) + 8 for k in range(len(SHAPES))]
        for k, s in enumerate(slots):
            assert np.array_equal(P.get_f(s), alone(k, dtype, P.time(s))), (dtype, mode, SHAPES[k])
