"""The forms of a time step agree.  A small lattice takes a step in one branch,
with the bulk cells in the boundary launch (automatic sweep grid); an explicit
grid takes it in two branches.  Both do the same arithmetic per cell and exact
sums per fiber, so every result has the same bits."""
import numpy as np
import pytest

from paper_1503_06869_amd import lbm

pytestmark = pytest.mark.gpu

WALLS = {
    "couette": dict(wall_u=0.03, init_couette=True),
    "periodic-force": dict(z_periodic=True, body_force=(1e-5, -2e-5, 3e-5)),
    "closed": dict(wall_u=0.02, x_walls=True, y_walls=True),
    "slip": dict(x_walls="free-slip", y_walls="free-slip", z_free_slip=True),
    "mixed": dict(x_walls="free-slip", y_walls=True, wall_u=0.01),
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


def run(shape, fibers, steps, grid, **kw):
    g = lbm.Context(*shape, tau=0.8, sweep_grid=grid, **kw)
    for X, q, l in fibers:
        g.add_fiber(np.array(X), np.array(q) / np.linalg.norm(q), l, 1.6, V=(0.01, -0.02, 0.015), W=(0.01, 0.02, -0.01),
                    force=(1e-3, 2e-3, -1e-3))
    for n in steps:
        g.step(n)
    out = (g.history(0, sum(steps)) if fibers else np.zeros(1),) + tuple(g.fields()) + (g.populations(),)
    g.close()
    return out


# 7 x 5 x 3: less than two waves of cells; 64 | ncell and not; close fibers,
# whose cells have links of both; the largest lattice of the rule and the
# smallest beyond it
CASES = [((7, 5, 3), [], "couette"),
         ((16, 12, 8), [([7.2, 6.1, 4.0], [1, 0.1, 0, 0], 4.5)], "couette"),
         ((21, 19, 23), [([4.0, 9.5, 11.2], [0.6, 0.1, 0.7, 0.2], 12.0), ([8.6, 10.0, 11.9], [0.6, 0.1, 0.7, 0.2], 12.0)],
          "periodic-force"),
         ((21, 18, 23), [([10.2, 9.5, 11.2], [0.5, 0.4, 0.1, 0.2], 9.0)], "closed"),
         ((20, 19, 23), [([10.2, 9.5, 11.2], [0.5, 0.4, 0.1, 0.2], 9.0)], "slip"),
         ((21, 19, 24), [([10.2, 9.5, 11.2], [0.5, 0.4, 0.1, 0.2], 9.0)], "mixed"),
         ((125, 125, 112), [([60.2, 59.5, 61.2], [0.5, 0.4, 0.1, 0.2], 19.0)], "couette"),
         ((125, 127, 112), [([60.2, 59.5, 61.2], [0.5, 0.4, 0.1, 0.2], 19.0)], "couette")]


@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "bf16"])
@pytest.mark.parametrize("shape,fibers,walls", CASES, ids=["%dx%dx%d-%s" % (c[0] + (c[2],)) for c in CASES])
def test_one_and_two_branches_agree(shape, fibers, walls, storage):
    if shape[0] > 100 and storage != "f32":
        pytest.skip("size rule: one storage suffices")
    a, b = (run(shape, fibers, (1, 22, 2), grid, storage=storage, **WALLS[walls]) for grid in (0, 37))
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert np.isfinite(a[-1]).all()


@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("shape,n", [((127, 126, 128), 1), ((163, 160, 162), 1), ((163, 160, 162), 16)])
def test_bulk_sweep_beside_the_branch(storage, shape, n):
    """16-bit storage: the workgroups of the bulk sweep that leave the particle
    branch room (small lattice; many fibers for the lattice) and those that do
    not (an explicit grid; few fibers) do the same arithmetic."""
    fibers = [([20.0 + 38.0 * (i % 4), 20.0 + 38.0 * (i // 4), 60.0], [0.5, 0.4, 0.1, 0.2], 24.0) for i in range(n)]
    a, b = (run(shape, fibers, (1, 6, 2), grid, storage=storage, **WALLS["couette"]) for grid in (0, 512))
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
