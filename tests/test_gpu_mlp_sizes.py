"""The network's passes at the sizes where their split changes: fewer samples
than a workgroup's waves, a tile of 32 and one more, more tiles than partial
sums (64), more samples than one pass through the work buffer (8192).
Against the FP64 reference: outputs and loss to 1e-5 (an FP32 chain of 375
multiply-adds), the gradient to 1e-4 of its norm (tiles of 32 samples and 64
partials in FP32 from deltas of 1e-5)."""
import numpy as np
import pytest

from oracle import closure_ref as R
from paper_1503_06869_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lbm.load()
    yield


@pytest.mark.parametrize("n", [1, 3, 32, 33, 2049, 8192, 8225])
def test_passes_match_reference(n):
    import torch
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, R.NI)).astype(np.float32)
    t = rng.standard_normal((n, R.NO)).astype(np.float32)
    m = lbm.Mlp(seed=5)
    w, _ = m.params()
    xd, td = torch.tensor(x, device="cuda"), torch.tensor(t, device="cuda")
    yd = torch.full((n + 1, R.NO), 7.0, device="cuda")
    m.forward(xd.data_ptr(), n, yd.data_ptr())
    y = yd.cpu().numpy()
    yr = R.forward(R.bf16_round(w), x.astype(np.float64))
    assert np.abs(y[:n] - yr).max() < 1e-5 * np.abs(yr).max() and (y[n] == 7.0).all()
    loss, grad = m.loss_grad(xd.data_ptr(), td.data_ptr(), n)
    lr, gr = R.loss_grad(R.bf16_round(w), x.astype(np.float64), t.astype(np.float64))
    assert abs(loss / lr - 1) < 1e-5 and np.linalg.norm(grad - gr) < 1e-4 * np.linalg.norm(gr)
    loss2, grad2 = m.loss_grad(xd.data_ptr(), td.data_ptr(), n)
    assert loss2 == loss and np.array_equal(grad2, grad)
    m.close()


def test_training_step_is_gradient_and_update():
    """One sample, one epoch: the same bits as the gradient and Adam called apart."""
    import torch
    rng = np.random.default_rng(2)
    xd = torch.tensor(rng.standard_normal((1, R.NI)).astype(np.float32), device="cuda")
    td = torch.tensor(rng.standard_normal((1, R.NO)).astype(np.float32), device="cuda")
    a, b = lbm.Mlp(seed=5), lbm.Mlp(seed=5)
    a.train(xd.data_ptr(), td.data_ptr(), 1, 1, 1, 1e-3)
    b.loss_grad(xd.data_ptr(), td.data_ptr(), 1)
    b.adam(1e-3, 0.9, 0.999, 1e-8)
    for p, q in zip(a.params(), b.params()):
        assert np.array_equal(p, q)
    a.close()
    b.close()
