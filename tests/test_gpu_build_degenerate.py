"""The builder on sites whose cells' faces nearly meet in one point: lattices
disturbed by about the rounding of their coordinates, points on circles about
one axis, points on spheres (whose bisectors all go through the centre, some
within their rounding of one line), far clusters. Against the oracle's brute-force faces, with the
tolerances of the other tests of volumes and faces: 1e-9 of the volume, faces
of more than 1e-9 of the cell's scale squared."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BOX = np.array([-1.0, -1, -1, 1, 1, 1])


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


def _check(vrt, sites):
    grid = vrt.build_grid(sites, BOX)
    rp, col = (t.cpu().numpy() for t in grid.neighbors())
    vol = grid.volumes().cpu().numpy()
    res, ref = oracle.faces(sites, BOX, np.arange(len(sites)), cap=1024)[:2]
    assert np.max(np.abs(vol - ref) / ref) <= 1e-9
    for i in range(len(sites)):
        nb, ar = res[i]
        real = {int(j) for j, a in zip(nb, ar) if a > 1e-9 * ref[i] ** (2 / 3)}
        assert real <= set(col[rp[i]:rp[i + 1]].tolist()), i


def _near_lattice(seed):
    r = np.random.default_rng(seed)
    r.random()
    n = int(r.integers(5, 9))
    m = (np.arange(n) + 0.5) / n * 2 - 1
    s = np.stack(np.meshgrid(m, m, m, indexing="ij"), -1).reshape(-1, 3)
    axis = r.integers(3)
    s[:, axis] += r.normal(size=len(s)) * 10 ** r.uniform(-16, -9)
    return s


def _circles(seed):
    r = np.random.default_rng(seed)
    n = int(70 * (900 / 70) ** r.random())
    a = r.uniform(0, 2 * np.pi, n)
    return np.stack([0.5 * np.cos(a), 0.5 * np.sin(a), r.choice(np.linspace(-0.9, 0.9, 7), n)], -1)


# Cells that degenerate in the loose order of the first pass (a vertex of
# three planes through one line), and do not when the planes come nearest first.
@pytest.mark.parametrize("sites,seed", [(_near_lattice, 591), (_near_lattice, 1167), (_near_lattice, 1467),
                                        (_circles, 570), (_circles, 738), (_circles, 822)])
def test_degenerate_in_the_loose_order(vrt, sites, seed):
    _check(vrt, sites(seed))


def _sphere(seed):
    r = np.random.default_rng(seed)
    d = r.normal(size=(1000 if seed % 2 else 100, 3))
    return 0.7 * d / np.linalg.norm(d, axis=1, keepdims=True)


def _spheres(seed):
    r = np.random.default_rng(seed)
    d = r.normal(size=(5, 200, 3))
    d *= np.array([0.1, 0.2, 0.4, 0.6, 0.8])[:, None, None] / np.linalg.norm(d, axis=2, keepdims=True)
    return d.reshape(-1, 3)


def _rounded_lattice(seed):
    r = np.random.default_rng(seed)
    n = int(r.integers(5, 9))
    m = (np.arange(n) + 0.5) / n * 2 - 1
    s = np.stack(np.meshgrid(m, m, m, indexing="ij"), -1).reshape(-1, 3)
    return s + r.normal(size=s.shape) * 10 ** r.uniform(-13, -11) * (r.random((len(s), 1)) < r.random())


# Cells that a cut leaves as no closed polyhedron with the tolerance of all cells.
@pytest.mark.parametrize("sites,seed", [(_sphere, 0), (_sphere, 1), (_sphere, 2), (_sphere, 3), (_spheres, 0), (_spheres, 1),
                                        (_spheres, 2), (_spheres, 3)] + [(_rounded_lattice, k) for k in range(6)])
def test_cells_are_closed(vrt, sites, seed):
    _check(vrt, sites(seed))


def _far_cluster(seed):
    r = np.random.default_rng(seed)
    n = int(np.exp(r.uniform(np.log(70), np.log(900)))) // 2
    size = 10 ** r.uniform(-6, -2)
    d = r.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return np.concatenate([size * d + r.uniform(-0.5, 0.5, 3), r.uniform(-1, 1, (n, 3))])


def _rounded_points(seed):
    r = np.random.default_rng(seed)
    n = int(np.exp(r.uniform(np.log(70), np.log(900))))
    s = np.unique(r.integers(-6, 7, (n, 3)) / 6.5, axis=0)
    return s + r.normal(size=s.shape) * 10 ** r.uniform(-16, -11)


def _few(seed):
    """At most 64 sites: all of a cell's planes come at once."""
    r = np.random.default_rng(seed)
    n = int(r.integers(8, 33))
    s = np.unique(r.integers(-3, 4, (2 * n, 3)) / 3.5, axis=0)
    return s + r.normal(size=s.shape) * 10 ** r.uniform(-16, -9)


# Cells that need their planes in the exact order of distance: planes of a far cluster's sites, nearly parallel, at
# distances equal to 2^-20; lattice points with distances equal to the disturbance of their coordinates.
@pytest.mark.parametrize("sites,seed", [(_far_cluster, 2349), (_rounded_points, 2012), (_rounded_points, 4604),
                                        (_few, 206), (_few, 3378)])
def test_planes_come_in_the_exact_order(vrt, sites, seed):
    _check(vrt, sites(seed))
