"""vor_locate where the walk along the neighbour table cannot be sure: points on
walls, edges and corners of the box, on faces, edges and vertices of lattice
cells, midway between sites; points that are sites; numbers of sites around the
least that walk. The cells are those of the definition, the lowest index among
the nearest sites, with squared distances as it computes them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


def _points(rng, sites, lo, hi):
    n, ext = 600, hi - lo
    u = lo + rng.random((n, 3)) * ext
    wall = u.copy()
    for a in range(3):
        k = rng.random(n)
        wall[k < 0.3, a] = lo[a]
        wall[k > 0.7, a] = hi[a]
    i, j = rng.integers(0, len(sites), (2, n))
    mid = 0.5 * (sites[i] + sites[j])
    grid = lo + np.round(rng.random((n, 3)) * 12) / 12 * ext
    near = sites[i] + 1e-13 * ext * rng.normal(size=(n, 3))
    return np.clip(np.concatenate([u, wall, sites[i], mid, grid, near]), lo, hi)


@pytest.mark.parametrize("case", ["n1", "n2", "n31", "n32", "n33", "n700", "lattice", "slab", "halo"])
def test_nearest_site_everywhere(vrt, case):
    rng = np.random.default_rng(sum(map(ord, case)))
    lo, hi = np.array([-1.0, -1, -1]), np.array([1.0, 1, 1])
    if case == "slab":
        lo, hi = np.array([-1000.0, -1, -0.01]), np.array([1000.0, 1, 0.01])
    if case[0] == "n":
        sites = rng.uniform(lo, hi, (int(case[1:]), 3))
    elif case == "lattice":
        m = (np.arange(6) + 0.5) / 3 - 1
        sites = rng.permutation(np.array([[x, y, z] for x in m for y in m for z in m]))
    elif case == "slab":
        sites = rng.uniform(lo, hi, (500, 3))
    else:
        sites = np.concatenate([0.01 * rng.normal(size=(800, 3)), rng.uniform(-1, 1, (20, 3))])
    pts = _points(rng, sites, lo, hi)
    got = vrt.locate(vrt.build_grid(sites, [*lo, *hi]), pts).cpu().numpy()
    d = pts[:, None, :] - sites[None, :, :]
    want = ((d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]).argmin(axis=1)   # the first of equals
    assert np.array_equal(got, want)
