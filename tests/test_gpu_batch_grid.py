"""The batched sweep's workgroups: one per 256 cells in FP32, a fixed number that
stride over them in 16-bit storage.  Two cases of 8790 chunks together, more
than the 8192 workgroups of the strided form on a card of 256 compute units,
have the bits of their single-lattice runs."""
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


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_many_chunks(storage):
    cases = scenarios.batched_cases(5, n_cases=2, edge=(104, 104))
    cases[1].nx += 1
    b = lbm.Batch(cases, storage=storage, history_capacity=64)
    b.step(5)
    for c, sc in enumerate(cases):
        g = single(sc, storage)
        g.step(5)
        assert_case_equal(b, c, g, 5)
        g.close()
    b.close()
