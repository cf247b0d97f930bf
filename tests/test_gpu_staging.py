"""Fields and populations read into host arrays: through the pinned ring
(pageable arrays, from 32 MiB), and by one copy (smaller reads, pinned
arrays), against the same values read on the device. The sizes lie around the
32 MiB and off the ring's chunks of 1 MiB. Values: bitwise."""
import ctypes
import threading

import numpy as np
import pytest

from gpu_util import smooth_random_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402

# sites: 9 doubles each of get_f, 3 of moments
SIZES = [(61, 37), (171, 170), (257, 255), (680, 685), (683, 683), (684, 684), (1024, 1024), (1182, 1184), (1031, 1019)]


def lattice(nx, ny, seed):
    L = lbm.Lattice(nx, ny, 0.7, 0.3, "f64")
    L.init(*smooth_random_state(nx, ny, seed=seed))
    return L.step(3)


def device_fields(L):
    d = torch.empty(3, L.ny, L.nx, dtype=torch.float64, device="cuda")
    L.moments_device(d[0], d[1], d[2])
    return d.cpu().numpy()


@pytest.mark.parametrize("nx,ny", SIZES)
def test_reads_equal_device_values(nx, ny):
    with lattice(nx, ny, 3) as L:
        want = device_fields(L)
        for _ in range(2):  # a new ring, then the kept one
            for a, b in zip(L.moments()[:3], want):
                assert np.array_equal(a, b)
        f = L.get_f()
        pinned = torch.empty(9, ny, nx, dtype=torch.float64, pin_memory=True)
        assert L._L.lbm_get_f(L._h, ctypes.c_void_p(pinned.data_ptr())) == 0
        assert np.array_equal(f, pinned.numpy())
        ys, xs = np.unravel_index(np.arange(0, nx * ny, max(1, nx * ny // 997)), (ny, nx))
        assert np.array_equal(L.sample_f(xs, ys), f[:, ys, xs].T)
        uy = np.zeros((ny, nx))  # one part only
        assert L._L.lbm_moments(L._h, None, None, uy.ctypes.data_as(ctypes.c_void_p), None) == 0
        assert np.array_equal(uy, want[2])


def test_reads_from_several_threads():
    lattices = [lattice(1250 + 13 * k, 1140 + 7 * k, k) for k in range(5)]
    want = [device_fields(L) for L in lattices]
    bad = []

    def read(L, w):
        for _ in range(4):
            L.step(0)
            got = L.moments()[:3]
            if not all(np.array_equal(a, b) for a, b in zip(got, w)):
                bad.append((L.nx, L.ny))

    team = [threading.Thread(target=read, args=a) for a in zip(lattices, want)]
    for t in team:
        t.start()
    for t in team:
        t.join()
    for L in lattices:
        L.close()
    assert not bad


def test_pool_reads():
    with lbm.Pool(1 << 28, "f32") as P:
        P.set_mode(lbm.GROUPED)
        slots = [P.add(nx, ny, 0.7, 0.3) for nx, ny in ((300, 290), (1300, 1200))]
        for s, (nx, ny) in zip(slots, ((300, 290), (1300, 1200))):
            P.init(s, *smooth_random_state(nx, ny, seed=nx))
        P.step(slots, 9)
        for s, (nx, ny) in zip(slots, ((300, 290), (1300, 1200))):
            f = P.get_f(s)
            rho = P.moments(s)[0]
            # sums of nine terms of order 1 in two orders: 16 roundings of double precision
            assert np.abs(f.sum(0) - rho).max() <= 16 * 2.0 ** -53 * 4 + 16 * 2.0 ** -24 * 4
