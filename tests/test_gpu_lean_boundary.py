"""FP64: the boundary launch in fewer registers, which follows a bulk sweep that
starts first, gives the same bits as the one with all of them.  A grid of more
workgroups starts the sweep second and takes the latter."""
import numpy as np
import pytest

from paper_1503_06869_amd import lbm

pytestmark = pytest.mark.gpu

WALLS = {
    "couette": dict(wall_u=0.03, init_couette=True),
    "periodic-force": dict(z_periodic=True, body_force=(1e-5, -2e-5, 3e-5)),
    "closed": dict(wall_u=0.02, x_walls=True, y_walls=True),
    "slip": dict(x_walls="free-slip", y_walls="free-slip", z_free_slip=True),
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


def run(shape, fibers, grid, **kw):
    g = lbm.Context(*shape, tau=0.8, storage="f64", sweep_grid=grid, **kw)
    for X, l in fibers:
        g.add_fiber(np.array(X), np.array([0.6, 0.1, 0.7, 0.2]) / np.sqrt(0.9), l, 1.6, V=(0.01, -0.02, 0.015),
                    W=(0.01, 0.02, -0.01), force=(1e-3, 2e-3, -1e-3))
    for n in (1, 14, 2):
        g.step(n)
    out = (g.history(0, 17),) + tuple(g.fields()) + (g.populations(),)
    g.close()
    return out


# cells over list capacity on both sides of 32, at the least and beyond; a
# fiber across the periodic seam; two so close that cells have links of both;
# walls from 4000000 cells on and below
CASES = [((41, 37, 27), [([20.2, 18.1, 13.3], 6.0)], "couette"),
         ((41, 37, 25), [([20.2, 18.1, 13.3], 6.0)], "couette"),
         ((59, 47, 61), [([1.2, 46.1, 30.3], 12.0), ([5.8, 46.6, 31.0], 12.0)], "periodic-force"),
         ((160, 157, 160), [([60.2, 59.5, 61.2], 19.0)], "closed"),
         ((160, 157, 160), [([60.2, 59.5, 61.2], 19.0)], "slip"),
         ((159, 156, 161), [([60.2, 59.5, 61.2], 19.0)], "slip")]


@pytest.mark.parametrize("shape,fibers,walls", CASES, ids=["%dx%dx%d-%s" % (c[0] + (c[2],)) for c in CASES])
def test_same_bits(shape, fibers, walls):
    a, b = (run(shape, fibers, grid, **WALLS[walls]) for grid in (64, 1500))
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert np.isfinite(a[-1]).all()
