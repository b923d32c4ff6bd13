"""Rays from one point. Small launches add up a block's tallies in LDS before
the caller's arrays: against the same rays repeated until the launch is one of
one ray per lane (tallies, sums in no fixed order, to 1e-12 of the largest, as
in the transport tests), below, at and above the least launch that does so, on
a grid of few cells (every block meets more than its table holds) and one of
many. Large launches of such rays take all the blocks that fit: against slices."""
import pytest

from paper_1310_1854_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vrt():
    from paper_1310_1854_amd import vrt as v
    v.load()
    return v


def _rays(n, seed, box, source=True):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d = torch.randn(n, 3, dtype=torch.float64, device="cuda", generator=gen)
    if source:
        o = torch.zeros_like(d) + torch.tensor([0.011, -0.007, 0.003], dtype=torch.float64, device="cuda")
    else:
        lo, hi = torch.tensor(box, dtype=torch.float64, device="cuda").reshape(2, 3)
        o = lo + torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=gen) * (hi - lo)
    return o.contiguous(), d, gen


@pytest.mark.parametrize("mode", ["fp64", "mixed"])
@pytest.mark.parametrize("M,n,source", [(200, 1023, True), (200, 1024, True), (200, 9000, True), (200, 9000, False),
                                        (20_000, 9000, True), (20_000, 1025, False)])
def test_tallies_of_small_launches(vrt, mode, M, n, source):
    import torch
    w = W.uniform_cube(M=M, N=10, seed=M)
    g = vrt.build_grid(w.sites, w.box)
    rho = torch.as_tensor(w.density, device="cuda")
    o, d, gen = _rays(n, 7, w.box, source)
    stop = -torch.log(1.0 - torch.rand(n, dtype=torch.float64, device="cuda", generator=gen))
    wgt = 0.5 + torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
    k = 100_000 // n + 1
    kw = dict(mode=mode, segments="none", kappa=2.0, tallies=True, persistent=True)
    for st in (None, stop):
        one = vrt.trace(g, o, d, rho, tau_stop=st, weight=wgt, **kw)
        many = vrt.trace(g, o.repeat(k, 1), d.repeat(k, 1), rho, tau_stop=None if st is None else st.repeat(k),
                         weight=wgt.repeat(k), **kw)
        for key in ("tau", "n_seg", "status"):
            assert torch.equal(one[key].repeat(k), many[key]), key
        for key in ("tally_len", "tally_abs"):
            assert float((one[key] - many[key] / k).abs().max()) <= 1e-12 * float(one[key].max()), key
    # the arrays are added to, and one of the two may be missing
    t = torch.full_like(rho, 3.0)
    b = vrt.TraceBuffers(n, counters=False)
    vrt.trace_into(g, o, d, rho, b, kappa=2.0, mode=mode, persistent=True, weight=wgt, tally_abs=t)
    ref = vrt.trace(g, o, d, rho, weight=wgt, **kw)["tally_abs"]
    assert float((t - 3.0 - ref).abs().max()) <= 1e-12 * (3.0 + float(ref.max()))


@pytest.mark.parametrize("mode,records", [("fp64", "fp32"), ("mixed", "fp32"), ("mixed", "compact")])
def test_large_launches(vrt, mode, records):
    import torch
    n = 300_100
    w = W.exp_disc(M=20_000, N=10, seed=5)
    g = vrt.build_grid(w.sites, w.box, records=records, block_lists=True)
    rho = torch.as_tensor(w.density, device="cuda")
    o, d, _ = _rays(n, 11, w.box)
    d[:64] = torch.nan          # a wave without paths
    for lf in (True, False):
        big = vrt.trace(g, o, d, rho, mode=mode, segments="none", persistent=True, ordered=True, locate_first=lf)
        for a in range(0, n, 30_000):
            b = min(n, a + 30_000)
            part = vrt.trace(g, o[a:b], d[a:b], rho, mode=mode, segments="none")
            for key in ("tau", "n_seg", "status"):
                assert torch.equal(part[key], big[key][a:b]), (key, a)
