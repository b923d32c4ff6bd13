"""The builder's cells at the edges of its kernels' ranges, against the
oracle's brute-force faces: sites below, at and past one Hilbert
neighbourhood (64), one run of the box tree (16) and one of its nodes (1024);
cells with more faces than a small cell holds (34), up to 200; sparse sites
around a dense ball; and lattices, which take the strict order. Tolerances
are those of the other tests of volumes and faces: 1e-9 of the volume, faces
of more than 1e-9 of the cell's scale squared."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BOX = np.array([-2.0, -2, -2, 2, 2, 2])


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


def _ball(rng, n, r):
    d = rng.normal(size=(n, 3))
    return d / np.linalg.norm(d, axis=1, keepdims=True) * r * rng.random((n, 1)) ** (1 / 3)


def _sites(case):
    rng = np.random.default_rng(1310 + sum(map(ord, case)))
    if case.startswith("n"):
        return rng.uniform(-2, 2, (int(case[1:]), 3))
    if case.startswith("shell"):            # one cell with as many faces as the number says
        d = rng.normal(size=(int(case[5:]), 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        return np.concatenate([[[0.01, 0.02, -0.01]], d])
    if case == "halo":                      # a dense ball seen from a few far sites
        return np.concatenate([_ball(rng, 1500, 0.05), rng.uniform(-2, 2, (30, 3))])
    m = (np.arange(9) + 0.5) / 9 * 4 - 2    # lattice
    return rng.permutation(np.array([[x, y, z] for x in m for y in m for z in m]))


@pytest.mark.parametrize("case", ["n2", "n16", "n17", "n63", "n64", "n65", "n66", "n129", "n1024", "n1025", "shell40",
                                  "shell70", "shell200", "halo", "lattice"])
def test_cells_vs_oracle_faces(vrt, case):
    sites = _sites(case)
    grid = vrt.build_grid(sites, BOX, block_lists=True)
    rp, col = (t.cpu().numpy() for t in grid.neighbors())
    vol, bb = grid.volumes().cpu().numpy(), grid.bboxes().cpu().numpy()
    res, ref, rbb = oracle.faces(sites, BOX, np.arange(len(sites)), cap=512, bboxes=True)
    assert np.max(np.abs(vol - ref) / ref) <= 1e-9
    ext = (rbb[:, 3:] - rbb[:, :3]).max(axis=1)
    assert np.max(np.abs(bb - rbb).max(axis=1) / ext) <= 1e-9
    for i in range(len(sites)):
        row = col[rp[i]:rp[i + 1]]
        got = set(row.tolist())
        assert len(got) == len(row)
        n_in = int((row >= 0).sum())
        assert np.all(np.diff(row[:n_in]) > 0) and np.all(row[n_in:] < 0)   # ascending, walls last
        nb, ar = res[i]
        real = {int(j) for j, a in zip(nb, ar) if a > 1e-9 * ref[i] ** (2 / 3)}
        assert real <= got, (i, real - got)
        assert got <= {int(j) for j in nb} if case != "lattice" else got == real, i
    if case.startswith("shell"):
        assert (col[rp[0]:rp[1]] >= 0).sum() == len(sites) - 1
