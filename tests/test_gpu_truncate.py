"""vor_grid_truncate_row keeps the first entries of a row in internal order, as
its header says (rows are stored nearest first), and the rows stay whole: both
modes trace the damaged grid alike. And the kernels of one ray per lane on
damaged grids, of which smaller launches, with a group of lanes per ray, run
others: the no-exit fallback in every mode and layout, with the density bound
to the grid or not, and rays that enter from outside, against slices of the
same rays."""
import numpy as np
import pytest

from paper_1310_1854_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


def _internal(vrt, grid, sites):
    """The internal index of every site: where rays that start at the sites start."""
    import torch
    o = torch.as_tensor(sites, device="cuda")
    b = vrt.TraceBuffers(len(sites))
    vrt.trace_into(grid, o, torch.ones_like(o), None, b)
    return b.start_cell.cpu().numpy()


def _rows(grid):
    rp, col = (t.cpu().numpy() for t in grid.neighbors())
    return [col[a:b][col[a:b] >= 0] for a, b in zip(rp[:-1], rp[1:])]


@pytest.mark.parametrize("records", ["fp32", "compact"])
def test_first_entries_in_internal_order(vrt, records):
    rng = np.random.default_rng(8)
    sites = rng.uniform(-1, 1, (400, 3))
    grid = vrt.build_grid(sites, [-1] * 3 + [1] * 3, records=records)
    internal, before = _internal(vrt, grid, sites), _rows(grid)
    cut = {}
    for s in rng.permutation(400)[:60]:
        for keep in (int(rng.integers(4, 9)), int(rng.integers(0, 5)), 6):   # the last changes nothing
            grid.truncate_row(int(s), keep)
            cut[int(s)] = min(keep, cut.get(int(s), 99))
    after = _rows(grid)
    for s in range(400):
        want = before[s]
        if s in cut:
            want = np.sort(want[np.argsort(internal[want])][: cut[s]])
        assert np.array_equal(after[s], want), s
    w = rng.normal(size=(2, 3000, 3))
    o = np.clip(0.5 * w[0], -1, 1)
    a, b = (vrt.trace(grid, o, w[1], None, mode=m, segments="exact", eps_fb=1e-3) for m in ("fp64", "mixed"))
    for k in ("n_seg", "n_fallback", "status", "seg_cell", "seg_len"):
        assert (a[k] == b[k]).all(), k
    assert int(a["n_fallback"].sum()) > 0


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("bound", [False, True])
@pytest.mark.parametrize("mode,records", [("fp64", "fp32"), ("mixed", "fp32"), ("mixed", "compact")])
def test_lane_kernels_on_damaged_grids(vrt, mode, records, bound, persistent):
    import torch
    n, few = 90_000, 10_000            # one ray per lane; a group of lanes per ray
    w = W.exp_disc(M=3_000, N=n, seed=12)
    g = vrt.build_grid(w.sites, w.box, records=records, block_lists=persistent)
    rng = np.random.default_rng(2)
    for s in rng.permutation(len(w.sites))[:300]:
        g.truncate_row(int(s), 4)
    rho = torch.as_tensor(w.density, device="cuda")
    o, d = (torch.as_tensor(x, device="cuda").clone() for x in (w.origins, w.dirs))
    o[: n // 3] += 30.0 * torch.sign(torch.randn(n // 3, 3, dtype=torch.float64, device="cuda",
                                                 generator=torch.Generator(device="cuda").manual_seed(1)))   # outside
    d[: n // 3] = torch.as_tensor(w.origins[: n // 3], device="cuda") - o[: n // 3]
    if bound:
        g.bind_density(rho)
    for enter in (False, True):
        kw = dict(mode=mode, segments="stride", seg_stride=160, grid_density=bound, persistent=persistent, ordered=persistent,
                  enter=enter, eps_fb=1e-4)
        r = None if bound else rho
        big = vrt.trace(g, o, d, r, **kw)
        assert int((big["n_fallback"] > 0).sum()) > 100
        inside = (big["status"] == vrt.RAY_OK)[: n // 3]
        assert int(inside.sum()) > (n // 4 if enter else -1) and (enter or not inside.any())
        for a in range(0, n, few):
            part = vrt.trace(g, o[a:a + few], d[a:a + few], r, **kw)
            for k in ("tau", "n_seg", "status", "n_fallback"):
                assert torch.equal(part[k], big[k][a:a + few]), (k, a, enter)
            c, ln = (big[k][160 * a:160 * (a + few)].view(few, 160) for k in ("seg_cell", "seg_len"))
            used = torch.arange(160, device="cuda")[None, :] < part["n_seg"][:, None]
            assert torch.equal(part["seg_cell"].view(few, 160)[used], c[used]) and \
                torch.equal(part["seg_len"].view(few, 160)[used], ln[used]), (a, enter)
