"""Sweeps with side or free-slip walls, whose odd form takes the waves at a wall
apart and lets a wave take another quarter of each chunk of cells: a few
workgroups with many chunks each, one workgroup per chunk and the one-branch
form give the same bits, for rows of whole waves, rows that straddle them and
a ragged last chunk."""
import numpy as np
import pytest

from paper_1503_06869_amd import lbm

pytestmark = pytest.mark.gpu

WALLS = {
    "closed": dict(wall_u=0.02, x_walls=True, y_walls=True),
    "slip": dict(x_walls="free-slip", y_walls="free-slip", z_free_slip=True),
    "z-slip": dict(z_free_slip=True, body_force=(1e-5, 2e-5, 0.0)),
    "mixed": dict(x_walls=True, y_walls="free-slip", wall_u=0.01),
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


def run(shape, grid, fiber, **kw):
    g = lbm.Context(*shape, tau=0.7, sweep_grid=grid, init_couette=True, **kw)
    if fiber:
        g.add_fiber(0.5 * np.array(shape), [0.8, 0.2, 0.4, 0.4], 5.0, 1.6, V=(0.01, -0.02, 0.015), force=(1e-3, 2e-3, -1e-3))
    else:
        u = np.random.default_rng(5).uniform(-1e-3, 1e-3, g.populations().shape)
        g.set_populations(u)
    g.step(7)
    out = g.populations()
    g.close()
    return out


@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "bf16"])
@pytest.mark.parametrize("shape", [(64, 12, 13), (128, 10, 11), (192, 7, 9), (41, 21, 19), (256, 5, 7)],
                         ids=lambda s: "%dx%dx%d" % s)
@pytest.mark.parametrize("walls", list(WALLS))
def test_grids_agree(walls, shape, storage):
    fiber = min(shape) > 11
    ref = run(shape, 100000, fiber, storage=storage, **WALLS[walls])
    assert np.isfinite(ref).all()
    for grid in (0, 3, 5):
        assert np.array_equal(run(shape, grid, fiber, storage=storage, **WALLS[walls]), ref)
