"""Mapping and boundary list on either side of the number of fibers from which
waves collect the cells to be tested: owners equal the FP64 predicate at the
fibers' poses, flags and the list's length follow from the owners, for both
shapes, close neighbours, fibers across the periodic seams, one too long for
the short cut by distance, and regions of more cells than a queue holds."""
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


C = [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1) if 0 < abs(x) + abs(y) + abs(z) < 3]


def owners(shape, per, X, q, L, r, kind):
    """Lowest fiber whose predicate holds at each cell centre (-1: fluid)."""
    nx, ny, nz = shape
    out = np.full((nz, ny, nx), -1, np.int32)
    grid = np.meshgrid(np.arange(nz, dtype=float), np.arange(ny, dtype=float), np.arange(nx, dtype=float), indexing="ij")[::-1]
    for p in reversed(range(len(X))):
        w, x, y, z = q[p]
        t = (1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y + w * z), 2.0 * (x * z - w * y))
        d = []
        for k, n in enumerate(shape):
            v = grid[k] - X[p][k]
            if k < 2 or per:
                v = np.where(v > 0.5 * n, v - n, np.where(v < -0.5 * n, v + n, v))
            d.append(v)
        a = d[0] * t[0] + d[1] * t[1] + d[2] * t[2]
        dist2 = (d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) - a * a
        if kind[p] == "spherocylinder":
            e = np.abs(a) - (0.5 * L[p] - r[p])
            inside = np.where(e <= 0.0, dist2 <= r[p] * r[p], dist2 + e * e <= r[p] * r[p])
        else:
            inside = (a * a <= (0.5 * L[p]) * (0.5 * L[p])) & (dist2 <= r[p] * r[p])
        out[inside] = p
    return out


def near(pid, per):
    solid = pid >= 0
    m = np.zeros_like(solid)
    for cx, cy, cz in C:
        s = np.roll(solid, (-cx, -cy), (2, 1))
        if per or cz == 0:
            s = np.roll(s, -cz, 0)
        else:
            z = np.zeros_like(s)
            z[max(0, -cz):s.shape[0] - max(0, cz)] = s[max(0, cz):s.shape[0] - max(0, -cz)]
            s = z
        m |= s
    return m & ~solid


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("per", [False, True], ids=["walls", "periodic"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 9])
def test_owners_flags_and_list(n, per, storage):
    shape = (44, 40, 46)
    g = lbm.Context(*shape, tau=0.8, z_periodic=per, storage=storage, **({} if per else dict(wall_u=0.02, init_couette=True)))
    rng = np.random.default_rng(n)
    X, L, r, kind = [], [], [], []
    # a long one (its half-length and radius plus three cells pass half the
    # shortest edge), then a lattice of short ones, some across the seams
    spots = [(22.3, 20.1, 23.4)] + [(x, y, z) for z in (7.2, 38.4) for x in (1.5, 12.7, 24.2, 33.9) for y in (3.3, 21.8)]
    for k in range(n):
        X.append(spots[k])
        L.append(34.0 if k == 0 else 7.0 + 0.3 * k)
        r.append(1.7 if k == 0 else 1.4 + 0.1 * k)
        kind.append("spherocylinder" if k % 2 else "cylinder")
        q = np.array([1.0, 0.0, 0.0, 0.05]) if k == 0 else np.array([1.0, 0.1, 0.15, 0.1]) * rng.choice([-1.0, 1.0], 4)
        g.add_fiber(X[k], q / np.linalg.norm(q), L[k], r[k], V=0.1 * rng.standard_normal(3), W=0.01 * rng.standard_normal(3),
                    shape=kind[k])
    for steps in (0, 1, 7):
        g.step(steps)
        Xn, qn = g.fiber_state()[:2]
        _, _, flags, pid = g.fields()
        want = owners(shape, per, Xn, qn, L, r, kind)
        assert np.array_equal(pid, want)
        m = near(want, per)
        assert np.array_equal(flags, (want >= 0).astype(np.uint8))
        assert g.info()["boundary_cells"] == m.sum()
    g.close()
