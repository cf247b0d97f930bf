"""The moments kernel (fields and totals in one launch) against sums over the
exported populations: widths around the lanes of a wave, where several rows
share one (up to 64 columns), around the columns of a segment, and with wrapped
columns at both ends; heights of one unit and with remainders. Both sides are
sums of at most nine FP64 terms below 1 in size, in two orders, a product with
the link and a division: 16 roundings; the shifted forms add one."""
import math

import numpy as np
import pytest

from gpu_util import smooth_random_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_0707_2437_amd as lbm  # noqa: E402

E = np.array([(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)], dtype=np.float64)
WIDTHS = [3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129, 255, 256, 257, 258, 260, 513]


def check(L, extra=1):
    f = L.get_f()
    rho, ux, uy, tot = L.moments()
    j = np.tensordot(E.T, f, axes=1)
    tol = 32 * extra * 2.0 ** -53
    assert np.abs(rho - f.sum(0)).max() <= tol
    assert np.abs(ux - j[0] / f.sum(0)).max() <= tol and np.abs(uy - j[1] / f.sum(0)).max() <= tol
    for k, a in enumerate((f, f * E[:, 0, None, None], f * E[:, 1, None, None])):
        assert abs(tot[k] - math.fsum(a.reshape(-1))) <= tol * np.abs(a).sum(), k
    assert np.array_equal(L.totals(), tot)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("ny", [3, 16, 67, 1029])
def test_moments_of_widths(dtype, ny):
    for nx in WIDTHS:
        with lbm.Lattice(nx, ny, 0.7, 0.3, dtype) as L:
            check(L.init(*smooth_random_state(nx, ny, seed=nx + ny)).step(2), 2 if dtype[-1] == "s" else 1)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(3, 100001), (5, 52429), (64, 4099), (40000, 3)])
def test_moments_of_long_lattices(dtype, nx, ny):
    with lbm.Lattice(nx, ny, 0.7, 0.3, dtype) as L:
        check(L.init(*smooth_random_state(nx, ny, seed=3)).step(2))


@pytest.mark.parametrize("nx,ny", [(5, 40), (64, 9), (130, 20), (700, 3)])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_a_non_finite_site_reaches_the_totals_and_no_other_site(nx, ny, value):
    with lbm.Lattice(nx, ny, 0.7, 0.3, "f64") as L:
        L.init(*smooth_random_state(nx, ny, seed=1))
        f = L.get_f()
        for y, x in ((0, 0), (ny - 1, nx - 1), (ny // 2, nx // 2)):
            g = f.copy()
            g[0, y, x] = value  # the rest population stays at its site
            L.set_f(g)
            with pytest.raises(lbm.LBMError) as e:
                L.moments()
            assert e.value.status == lbm.ENONFINITE
            rho = L.moments(check=False)[0]
            assert not np.isfinite(rho[y, x]) and np.isfinite(rho).sum() == nx * ny - 1
