"""Launches of both kinds over the same rays: one launch large enough for one
ray per lane against slices small enough for a group of lanes per ray. Every
output is equal bit for bit (the tallies, sums in no fixed order, to 1e-12 of
the largest, as in the transport tests)."""
import numpy as np
import pytest

from paper_1310_1854_amd import workloads as W

pytestmark = pytest.mark.gpu

N = 262_200         # past the largest launch with groups (262144 rays: FP64 without segments)
CUTS = [0, 1, 64, 1000] + list(range(32_768, N, 32_768)) + [N]       # slices of 1 to 32768 rays
SLICES = list(zip(CUTS[:-1], CUTS[1:]))


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


@pytest.fixture(scope="module")
def case(vrt):
    import torch
    w = W.exp_disc(M=20_000, N=N, seed=71)
    o, d = torch.as_tensor(w.origins, device="cuda"), torch.as_tensor(w.dirs, device="cuda")
    o[5], d[6], d[7] = 99.0, 0.0, float("nan")       # no path: outside, no direction
    o[8, 0], d[8] = 10.0, torch.tensor([1.0, 0, 0])  # on the wall, heading out
    rho = torch.as_tensor(w.density, device="cuda")
    grids = {r: vrt.build_grid(w.sites, w.box, block_lists=(r == "fp32"), records=r) for r in ("fp32", "compact")}
    return grids, o.contiguous(), d.contiguous(), rho


@pytest.mark.parametrize("stride", [0, 5, 8, 16, 24, 64])
@pytest.mark.parametrize("mode,records", [("fp64", "fp32"), ("mixed", "fp32"), ("mixed", "compact")])
def test_group_and_lane_launches_agree(vrt, case, mode, records, stride):
    import torch
    grids, o, d, rho = case
    g = grids[records]
    kw = dict(mode=mode, segments="exact" if stride else "none", seg_stride=stride or 64,
              persistent=stride != 5, ordered=stride > 8, locate_first=stride != 24)
    big = vrt.trace(g, o, d, rho, **kw)
    at = 0
    counters = torch.zeros_like(big["counters"])
    for a, b in SLICES:
        part = vrt.trace(g, o[a:b], d[a:b], rho, **kw)
        for k in ("tau", "n_seg", "status", "n_fallback"):
            assert torch.equal(part[k], big[k][a:b]), (k, a)
        counters += part["counters"]
        if stride:
            n = int(part["ray_off"][-1])
            for k in ("seg_cell", "seg_len"):
                assert torch.equal(part[k][:n], big[k][at:at + n]), (k, a)
            at += n
    # (the steps re-decided in FP64 depend on how many planes a search looks at before it stops)
    same = [0, 1, 3, 4]
    assert torch.equal(counters[same], big["counters"][same])
    assert (counters[2] > 0) == (big["counters"][2] > 0) == (mode == "mixed")


@pytest.mark.parametrize("mode", ["fp64", "mixed"])
def test_group_transport_agrees(vrt, case, mode):
    import torch
    grids, o, d, rho = case
    g = grids["fp32"]
    gen = torch.Generator(device="cuda").manual_seed(5)
    stop = -torch.log(1.0 - torch.rand(N, dtype=torch.float64, device="cuda", generator=gen))
    stop[10:20] = 0.0
    stop[20:30] = float("nan")
    wgt = 0.5 + torch.rand(N, dtype=torch.float64, device="cuda", generator=gen)
    kw = dict(mode=mode, segments="stride", seg_stride=24, spill_chunks=4 * N, kappa=3.0, tallies=True, persistent=True,
              enter=True)
    big = vrt.trace(g, o, d, rho, tau_stop=stop, weight=wgt, **kw)
    tl, ta = torch.zeros_like(rho), torch.zeros_like(rho)
    for a, b in SLICES:
        part = vrt.trace(g, o[a:b], d[a:b], rho, tau_stop=stop[a:b], weight=wgt[a:b], **kw)
        for k in ("tau", "n_seg", "status", "stop_cell", "stop_s"):
            assert torch.equal(part[k], big[k][a:b]), (k, a)
        tl += part["tally_len"]
        ta += part["tally_abs"]
    for mine, ref in ((tl, big["tally_len"]), (ta, big["tally_abs"])):
        assert float((mine - ref).abs().max()) <= 1e-12 * float(ref.max())


def test_group_spill_runs_out(vrt, case):
    """A spill too small: counts and depths complete, the paths past it
    reported, and the chunks asked for counted."""
    import torch
    grids, o, d, rho = case
    ref = vrt.trace(grids["fp32"], o[:2000], d[:2000], rho, mode="fp64", segments="none")
    part = vrt.trace(grids["fp32"], o[:2000], d[:2000], rho, mode="fp64", segments="stride", seg_stride=8, spill_chunks=3)
    assert torch.equal(part["tau"], ref["tau"]) and torch.equal(part["n_seg"], ref["n_seg"])
    long = (part["n_seg"] > 8).cpu().numpy()
    over = (part["status"] == vrt.RAY_OVERFLOW).cpu().numpy()
    assert int(part["work"][2]) == long.sum() and np.all(long[over]) and long.sum() - over.sum() <= 3 and over.any()


def _odd_grid(name, rng):
    box = np.array([-1.0, -1, -1, 1, 1, 1])
    if name == "shell":       # one cell with 180 faces
        d = rng.normal(size=(180, 3))
        return np.concatenate([[[0.01, 0.0, 0.02]], 0.7 * d / np.linalg.norm(d, axis=1, keepdims=True)]), box
    if name == "halo":        # rows that mix near and very far neighbours
        return np.concatenate([0.02 * rng.normal(size=(1500, 3)), rng.uniform(-1, 1, (60, 3))]), box
    g = (np.arange(6) + 0.5) / 3 - 1   # lattice
    return rng.permutation(np.array([[x, y, z] for x in g for y in g for z in g])), box


@pytest.mark.parametrize("records", ["fp32", "compact"])
@pytest.mark.parametrize("name", ["shell", "halo", "lattice"])
def test_searches_that_stop_agree_with_whole_rows(vrt, name, records):
    """One ray per lane (searches that stop where the rest of a row is out of
    reach) against groups (whole rows), in both modes, on rows of very uneven
    neighbours and on a lattice, with rays along its planes, edges and
    diagonals."""
    import torch
    rng = np.random.default_rng(len(name))
    sites, box = _odd_grid(name, rng)
    n = 100_000
    o = rng.uniform(-1, 1, (n, 3))
    d = rng.normal(size=(n, 3))
    k = n // 4
    o[:k] = np.round(o[:k] * 6) / 6                                  # lattice points, edges and faces
    d[:k] = rng.integers(-1, 2, (k, 3)) + (rng.random((k, 1)) < 0.2) * 1e-9 * rng.normal(size=(k, 3))
    d[~d.any(axis=1)] = 1.0
    o[k:2 * k] = sites[rng.integers(0, len(sites), k)]
    grid = vrt.build_grid(sites, box, records=records)
    rho = torch.as_tensor(rng.random(len(sites)), device="cuda")
    o, d = torch.as_tensor(o, device="cuda"), torch.as_tensor(d, device="cuda")
    got = {m: vrt.trace(grid, o, d, rho, mode=m, segments="exact", persistent=True, ordered=True) for m in ("fp64", "mixed")}
    at = 0
    for a in range(0, n, 32_768):
        b = min(n, a + 32_768)
        part = vrt.trace(grid, o[a:b], d[a:b], rho, mode="fp64", segments="exact")
        m = int(part["ray_off"][-1])
        for big in got.values():
            for key in ("tau", "n_seg", "status"):
                assert torch.equal(part[key], big[key][a:b]), key
            for key in ("seg_cell", "seg_len"):
                assert torch.equal(part[key][:m], big[key][at:at + m]), key
        at += m
