"""Histories read in one piece (beyond the staging buffer's 256 KiB), in small
pieces (through it) and across the end of the ring are the same rows; windows
that the ring no longer holds stay refused."""
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


def context(**kw):
    g = lbm.Context(20, 16, 16, tau=0.8, wall_u=0.02, init_couette=True, **kw)
    g.add_fiber([9.3, 8.1, 7.7], [0.9, 0.1, 0.3, 0.2], 6.0, 1.4)
    return g


def test_large_and_small_reads_agree():
    g = context()
    g.step(2000)
    h = g.history(0, 2000)                       # 304 kB
    assert np.array_equal(h, np.concatenate([g.history(a, 500) for a in range(0, 2000, 500)]))
    F, M = g.force_torque()
    assert np.array_equal(h[-1, 0, :6], np.concatenate([F[0], M[0]]))
    g.close()


@pytest.mark.parametrize("first,count", [(11, 7), (12, 3), (13, 1), (14, 4), (13, 5), (17, 1), (14, 0)])
def test_windows_across_the_rings_end(first, count):
    case = scenarios.batched_cases(1, n_cases=2, edge=(20, 24))
    g, full = context(history_capacity=7), context()
    b, bfull = lbm.Batch(case, history_capacity=7), lbm.Batch(case)
    for x in (g, full, b, bfull):
        x.step(18)
    assert np.array_equal(g.history(first, count), full.history(first, count))
    assert np.array_equal(b.history(1, first, count), bfull.history(1, first, count))
    for bad in ((10, 1), (-1, 1), (16, 3)):
        with pytest.raises(lbm.LBMError):
            g.history(*bad)
        with pytest.raises(lbm.LBMError):
            b.history(1, *bad)
    for x in (g, full, b, bfull):
        x.close()
