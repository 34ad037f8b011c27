"""Steps of a batch taken in any grouping: single steps at odd and even counts
and replayed pairs give each case the bits of its single-lattice run, for
cases whose cells end inside a 256-cell chunk or with one, whose sweep chunks
and boundary workgroups lie among those of cases of other sizes."""
import numpy as np
import pytest

from paper_1503_06869_amd import lbm, scenarios

from test_gpu_batched import assert_case_equal, single

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


@pytest.mark.parametrize("storage,threads,bins", [("f32", 0, 0), ("f64", 256, 3), ("bf16", 1024, 2), ("f16", 512, 6)])
def test_any_grouping_of_steps(storage, threads, bins):
    cases = scenarios.batched_cases(11, n_cases=6, edge=(20, 36))
    for sc, n in zip(cases, ((32, 24, 32), (64, 32, 24), (25, 31, 27))):   # whole chunks twice, then a ragged end
        f = sc.fibers[0]
        f.X = np.asarray(f.X) * np.array(n) / (sc.nx, sc.ny, sc.nz)
        f.length, f.q = 9.0, np.array([1.0, 0.1, 0.2, 0.0]) / np.sqrt(1.05)
        f.X[2] = 0.5 * n[2]
        sc.nx, sc.ny, sc.nz = n
    groups = (1, 1, 2, 3, 4, 1, 5)
    b = lbm.Batch(cases, storage=storage, threads=threads, bins=bins)
    for n in groups:
        b.step(n)
    for c, sc in enumerate(cases):
        g = single(sc, storage)
        g.step(sum(groups))
        assert_case_equal(b, c, g, sum(groups))
        g.close()
    b.close()
