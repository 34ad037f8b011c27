"""Ends of the ranges of the forms: a coupled step on boxes of a few waves of
cells, the last one ragged, in one branch and in two; slender-body systems just
beyond the one-workgroup form and with more than 128 quadrature points, against
the FP64 reference (to which the device solves agree to 1e-10)."""
import numpy as np
import pytest

from oracle import sbf_ref as S
from paper_1503_06869_amd import lbm, scenarios

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


def coupled(shape, grid, storage):
    g = lbm.Context(*shape, tau=0.8, wall_u=0.01, init_couette=True, storage=storage, sweep_grid=grid)
    g.add_fiber(0.5 * (np.array(shape) - 1) + 0.1, [1.0, 0.1, 0.2, 0.1] / np.sqrt(1.06), 1.4, 0.55, 4.0, V=(0.01, -0.01, 0.005))
    g.step(9)
    out = (g.history(0, 9),) + tuple(g.fields()) + (g.populations(),)
    g.close()
    return out


@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "bf16"])
@pytest.mark.parametrize("shape", [(6, 5, 5), (7, 6, 6), (8, 8, 6)], ids=lambda s: "%dx%dx%d" % s)   # 3 waves; 4; 6 whole
def test_smallest_coupled_boxes(shape, storage):
    one, two = coupled(shape, 0, storage), coupled(shape, 1, storage)
    assert np.isfinite(one[-1]).all() and (one[3] > 0).any()
    for a, b in zip(one, two):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("m,N,nq", [(7, 5, 16), (11, 5, 8), (5, 2, 48), (3, 1, 64), (24, 2, 45)])
def test_sbf_beyond_the_one_workgroup_form(m, N, nq):
    from paper_1503_06869_amd import sbf
    rng = np.random.default_rng(m)
    L, eps = 48.0, 1 / 12.0
    sc = scenarios.sbf_cloud(seed=m, m=m, length=L, eps=eps, spacing=1.2)
    F = sc.F + 0.3 * rng.standard_normal((m, 3))
    Mt = 5.0 * np.cross(sc.p, rng.standard_normal((m, 3)))
    _, V_o, W_o = S.SBF(L, eps, N=N, nq=nq).solve(sc.X, sc.p, F, Mt)
    for launches in (False, True):
        g = sbf.SBF(m, L, eps, nmodes=N, nq=nq, gmres_tol=1e-13)
        g.enable_timing(launches)
        g.set_fibers(sc.X, sc.p, F, Mt)
        g.solve()
        V, W = g.velocities()
        g.close()
        assert np.abs(V - V_o).max() <= 1e-10 * np.abs(V_o).max()
        assert np.abs(W - W_o).max() <= 1e-10 * np.abs(W_o).max()
