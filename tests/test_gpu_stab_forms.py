"""Momentum stabilization in the two forms of a step: one branch (small
lattice, automatic grid) and two (explicit grid).  The forms add the same
momenta in other orders, so the means agree to the rounding of the sums and
the fields to what that moves; and the sums that one workgroup adds up at the
end of a step are few, whatever the lattice."""
import numpy as np
import pytest

from paper_1503_06869_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


def run(shape, grid, steps, **kw):
    g = lbm.Context(*shape, tau=0.8, sweep_grid=grid, stabilize=True, **kw)
    c = 0.5 * np.array(shape)
    q = np.array([0.5, 0.4, 0.1, 0.2])
    for s in (-1.0, 1.0):
        g.add_fiber(c + np.array([3.6 * s, 0.2, 0.3]), q / np.linalg.norm(q), 8.0, 1.6, force=(1e-3, 2e-3, -3e-3))
    means = []
    for n in steps:
        g.step(n)
        means.append(g.mean_velocity()[0])
    out = np.array(means), g.history(0, sum(steps)), g.populations()
    g.close()
    return out


# Waves of one round, two and three (1536 x 64 cells a round), the last
# ragged; walls beside the periodic axis.  FP64: a thread's cells, the
# waves and the slots are added in chains of fewer than 100 terms, so the two
# means differ by less than 100 x 1.1e-16 of the mean speed, below 0.02: 2e-16
# a step, and the fields follow it.  The exchange sums are rounded to 2^-46 =
# 1.4e-14 a link (2^-52 for the force), a few hundred links of a step may
# round the other way: 1e-11 of torque, which the moment of inertia of some
# 2000 turns into 1e-14 of spin.  1e-10 bounds the history, 1e-12 the rest.
@pytest.mark.parametrize("shape,kw", [((20, 18, 22), dict(z_periodic=True)), ((51, 50, 52), dict(z_periodic=True)),
                                      ((64, 61, 63), dict(z_periodic=True)),
                                      ((52, 51, 53), dict(z_periodic=True, x_walls="free-slip", y_walls=True)),
                                      ((54, 51, 53), dict(wall_u=0.01, init_couette=True))])
def test_forms_agree_with_stabilization(shape, kw):
    (ma, ha, fa), (mb, hb, fb) = (run(shape, grid, (1, 6, 2), storage="f64", **kw) for grid in (0, 37))
    assert np.isfinite(fa).all() and np.abs(ma).max() > 1e-9
    assert np.abs(ma - mb).max() <= 1e-12
    assert np.abs(fa - fb).max() <= 1e-12
    assert np.abs(ha - hb).max() <= 1e-10


# 32 bytes a slot, beside 1024 slots of the pass after set-up at least and the
# list of changed cells (4097 words without fibers)
@pytest.mark.parametrize("n", [32, 64, 96, 119])
def test_few_slots_on_small_lattices(n):
    extra = []
    for on in (True, False):
        g = lbm.Context(n, n, n, z_periodic=True, stabilize=on)
        extra.append(g.info()["device_bytes"])
        g.close()
    assert extra[0] - extra[1] <= 32 * 2048 + 4 * 4097 + 64
