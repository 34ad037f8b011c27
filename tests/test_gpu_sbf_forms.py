"""The two forms of the slender-body solve agree: whole steps of a few fibers
in one workgroup (everything in LDS), and the kernels in launches of their own
(taken with the event timing on, which brackets single kernels).  Both solve
the same system to a relative residual of 1e-13 with sums in other orders, so
velocities and positions agree to 1e-10 of their size.  Sizes: one fiber, the
smallest rules, several pairs per chunk of moments, restarts inside the solve,
and the largest systems on either side of the LDS limit."""
import numpy as np
import pytest

from paper_1503_06869_amd import lbm, scenarios

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


@pytest.mark.parametrize("m,N,nq,restart", [(1, 5, 16, 30), (2, 1, 1, 30), (2, 5, 16, 30), (2, 8, 20, 30), (3, 8, 5, 4),
                                            (4, 2, 40, 30), (5, 5, 16, 30), (6, 3, 8, 63), (9, 2, 7, 30), (7, 5, 16, 30)])
def test_one_workgroup_and_many_launches_agree(m, N, nq, restart):
    from paper_1503_06869_amd import sbf
    rng = np.random.default_rng(100 * m + N)
    L, eps = 48.0, 1 / 12.0
    if m == 2:
        sc = scenarios.sbf_pair(dist=15.1, tilt=0.1)
    else:
        sc = scenarios.sbf_cloud(seed=m, m=m, length=L, eps=eps, spacing=1.3)
    F = sc.F + 0.2 * rng.standard_normal((m, 3))
    Mt = 3.0 * np.cross(sc.p, rng.standard_normal((m, 3)))
    out = []
    for launches in (False, True):
        g = sbf.SBF(m + 1, L, eps, nmodes=N, nq=nq, gmres_tol=1e-13, gmres_restart=restart, gmres_maxit=400)
        g.set_fibers(sc.X, sc.p, F, Mt)
        g.enable_timing(launches)
        g.solve()
        V0, W0 = g.velocities()
        g.step(3, 2.0)
        g.step(2, 2.0)
        out.append([V0, W0, g.coefficients(), *g.velocities(), *g.state()])
        assert g.stats()["steps"] == 5
        g.close()
    for k, (x, y) in enumerate(zip(*out)):
        scale = np.abs(y).max()
        assert np.isfinite(x).all() and np.abs(x - y).max() <= 1e-10 * max(scale, 1e-30), (k, np.abs(x - y).max(), scale)
