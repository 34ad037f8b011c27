"""Lines of the batched form's tuning cache serve the batches that they were
timed for: equal lattices with longer, thicker or rounded fibers, another
storage, and lines of an earlier layout of the step (keyed by the lattices
alone) are timed anew; the same batch is not."""
import struct

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


def batch_cases():
    cases = scenarios.batched_cases(4, n_cases=3, edge=(28, 30))
    for sc in cases:
        f = sc.fibers[0]
        f.X, f.q, f.length, f.radius = [0.5 * sc.nx, 0.5 * sc.ny, 0.5 * sc.nz], [1.0, 0.1, 0.0, 0.0], 8.0, 2.0
    return cases


def tuned(path, change=None, **kw):
    cases = batch_cases()
    if change:
        change(cases[1].fibers[0])
    b = lbm.Batch(cases, **kw)
    t = b.autotune(trial_steps=1, cache_path=str(path))
    b.close()
    return t


def longer(f):
    f.length = 10.0


def thicker(f):
    f.radius = 2.5


def rounded(f):
    f.shape = "spherocylinder"


@pytest.mark.parametrize("change,kw", [(longer, {}), (thicker, {}), (rounded, {}), (None, {"storage": "f16"})],
                         ids=["longer", "thicker", "rounded", "storage"])
def test_other_work_is_timed_anew(tmp_path, change, kw):
    path = tmp_path / "cache.txt"
    assert tuned(path)["from_cache"] == 0
    assert tuned(path)["from_cache"] == 1
    assert tuned(path, change, **kw)["from_cache"] == 0


def test_lines_of_the_earlier_layout_are_not_taken(tmp_path):
    path = tmp_path / "cache.txt"
    tuned(path)
    head, cu, n, _ = path.read_text().split()[0].rsplit("-", 3)
    h = 1469598103934665603
    for byte in b"".join(struct.pack("<3i", sc.nx, sc.ny, sc.nz) for sc in batch_cases()) + struct.pack("<i", lbm.LBM_F32):
        h = ((h ^ byte) * 1099511628211) % 2 ** 64
    path.write_text("%s-%s-%s-%016x 1024 1 9.5\n" % (head.replace("v2-", "", 1), cu, n, h))
    assert tuned(path)["from_cache"] == 0
