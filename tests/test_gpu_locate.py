"""vor_locate's walk along the neighbour table against the oracle's brute
force, where it starts and where it must hand over to the search: site counts
around the steps of its start table (powers of 8), points at sites, on walls,
edges and corners of the box, on the bisector between two neighbours and a
rounding away from it, at lattice vertices, in a dense ball and its halo; and
grids whose neighbour table has been cut."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BOX = np.array([-2.0, -1, -2, 2, 3, 2])


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


def _sites(case, rng):
    if case.startswith("n"):
        return rng.uniform(BOX[:3], BOX[3:], (int(case[1:]), 3))
    if case == "halo":
        d = rng.normal(size=(2500, 3)) * 0.003 + [0.4, 0.3, 0.2]
        return np.concatenate([d, rng.uniform(BOX[:3], BOX[3:], (40, 3))])
    if case == "pairs":                     # sites 1e-7 apart, far from the others
        p = rng.uniform(BOX[:3] + 0.1, BOX[3:] - 0.1, (60, 3))
        return np.concatenate([p, p + 1e-7 * rng.normal(size=p.shape)])
    g = np.stack(np.meshgrid(*[BOX[a] + (np.arange(8) + 0.5) * 0.5 for a in range(3)], indexing="ij"), -1)
    return rng.permutation(g.reshape(-1, 3))


@pytest.mark.parametrize("case", ["n1", "n2", "n7", "n8", "n9", "n64", "n65", "n513", "n4097", "halo", "pairs", "lattice"])
def test_locate_vs_oracle(vrt, case):
    rng = np.random.default_rng(99 + sum(map(ord, case)))
    s = _sites(case, rng)
    a, b = s[rng.integers(0, len(s), 2000)], s[rng.integers(0, len(s), 2000)]
    mid = 0.5 * (a + b)
    wall = rng.uniform(BOX[:3], BOX[3:], (1500, 3))
    ax = rng.integers(0, 3, 1500)
    wall[np.arange(1500), ax] = np.where(rng.random(1500) < 0.5, BOX[ax], BOX[ax + 3])
    corner = np.array([[x, y, z] for x in BOX[[0, 3]] for y in BOX[[1, 4]] for z in BOX[[2, 5]]])
    vert = BOX[:3] + 0.5 * rng.integers(0, 9, (1500, 3))           # the lattice's cell corners
    near = s[rng.integers(0, len(s), 1500)] + 0.01 * rng.normal(size=(1500, 3))
    pts = np.concatenate([rng.uniform(BOX[:3], BOX[3:], (6000, 3)), s, mid, np.nextafter(mid, a), np.nextafter(mid, b),
                          wall, corner, vert, near, [[9.0, 0, 0], [np.nan, 0, 0]]])
    want, _ = oracle.locate(s, BOX, pts)
    grid = vrt.build_grid(s, BOX)
    assert np.array_equal(vrt.locate(grid, pts).cpu().numpy(), want)
    for n in (1, 63, 65):
        assert np.array_equal(vrt.locate(grid, pts[:n]).cpu().numpy(), want[:n])
    if len(s) > 100:
        for i in range(0, len(s), 7):
            grid.truncate_row(i, 2)
        assert np.array_equal(vrt.locate(grid, pts).cpu().numpy(), want)
