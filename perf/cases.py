"""The work that programs have this library do, as cases that can be timed.

Each case is one call (or one short sequence of calls) through the public
binding, ``paper_1310_1854_amd.vrt``, on a grid and rays of the shapes that
the repository's workloads use: a uniform cube, an exponential disc, a flared
disc and a clumpy medium. Inputs are drawn on the GPU from a seed.

  paths      vrt.trace_into into windows and spill chains, vrt.exclusive_scan and vrt.gather_paths: every ray's whole
             path as a compact row, with its optical depth
  windows    vrt.trace_into into kept buffers: a window of segments per ray, wide enough for nearly every path
  depth      vrt.trace_into into kept buffers: optical depths and segment counts alone
  transport  vrt.trace with interaction points and both per-cell tallies
  build      vrt.build_grid, the neighbour lists and the cell volumes of the new grid, and its release
  locate     vrt.locate or vrt.locate_blocks: the cell of each point
  serve      requests of mixed size and precision through vrt.Server, their paths copied out
"""
import math

import torch

from paper_1310_1854_amd import vrt

DEV = "cuda"
F64 = torch.float64
PER_RAY = 0.70         # cells a path crosses, per cube root of the site count (0.66 to 1.0 over the shapes)
NEIGHBOURS = 15.54     # neighbours of a cell of random sites (Sect. 2.1)
STRIDE = 128           # segments per window of the paths case


def listed():
    return [
        # a handful of rays, as an interactive probe or a peel-off towards one observer sends: latency alone
        dict(name="windows_61_exp_disc", op="windows", shape="exp_disc", M=100_000, N=61, mode="mixed", ordered=False,
             bound=False),
        # the FP64 correctness configuration: a small batch on a small grid, buffers kept
        dict(name="windows_1e4_cube_fp64", op="windows", shape="cube", M=1_000, N=10_000, mode="fp64", ordered=True,
             bound=False),
        # a batch of the size that the serving mix sends, traced directly, mixed precision
        dict(name="depth_20011_flared", op="depth", shape="flared_disc", M=1_000_000, N=20_011, mode="mixed",
             ordered=True, bound=True),
        # the exponential disc: a million packages from random sites
        dict(name="paths_1e6_exp_disc", op="paths", shape="exp_disc", M=100_000, N=1_000_000, mode="mixed",
             ordered=True, bound=True),
        # the flared disc at full size, half of the packages from the central source
        dict(name="paths_8e6_flared", op="paths", shape="flared_disc", M=1_000_000, N=8_000_000, mode="mixed",
             ordered=True, bound=True),
        # the same disc in double precision throughout, the density as a per-call array
        dict(name="paths_2e6_flared_fp64", op="paths", shape="flared_disc", M=1_000_000, N=2_000_003, mode="fp64",
             ordered=True, bound=False),
        # the clumpy medium, whose cell blocks exceed the last-level cache (compact records): the largest
        dict(name="paths_5e6_clumpy", op="paths", shape="clumpy", M=4_000_000, N=5_000_000, mode="mixed",
             ordered=True, bound=True),
        # Monte Carlo transport: packages stop at drawn depths and deposit in every cell they cross
        dict(name="transport_2e6_flared", op="transport", shape="flared_disc", M=1_000_000, N=2_000_000, mode="mixed",
             ordered=True, bound=True),
        # setup of a small grid, as a parameter scan repeats it
        dict(name="build_1e4_cube", op="build", shape="cube", M=10_000, blocks=False),
        # setup of the flared disc with the block lists
        dict(name="build_1e6_flared", op="build", shape="flared_disc", M=1_000_000, blocks=True),
        # the grid-quality measure: the cells of points uniform over the box, by the bucket grid
        dict(name="locate_5e6_flared", op="locate", shape="flared_disc", M=1_000_000, N=5_000_000, blocks=False),
        # continuous serving of requests of 256 to 65536 rays over three resident grids
        dict(name="serve_12_mixed", op="serve", scale=1.0, lo=256, hi=65_536),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["paths", "paths", "paths", "windows", "depth", "transport", "build", "build", "locate", "locate",
                     "serve"])
    if op == "serve":
        lo = log(64, 1024)
        return dict(op=op, scale=round(rng.uniform(0.05, 1.0), 3), lo=lo, hi=log(4 * lo, 65_536))
    shape = rng.choice(["cube", "exp_disc", "flared_disc", "clumpy"])
    top = {"cube": 300_000, "exp_disc": 500_000, "flared_disc": 1_500_000, "clumpy": 4_000_000}[shape]
    if op == "build":
        return dict(op=op, shape=shape, M=log(1_000, min(top, 1_500_000)), blocks=rng.random() < 0.5)
    M = log(1_000, top)
    if op == "locate":
        return dict(op=op, shape=shape, M=M, N=log(1, 5_000_000), blocks=rng.random() < 0.5)
    N = log(1, {"paths": 4_000_000, "windows": 200_000, "depth": 4_000_000, "transport": 2_000_000}[op])
    return dict(op=op, shape=shape, M=M, N=N, mode=rng.choice(["mixed", "mixed", "fp64"]), ordered=N > 4096 or
                rng.random() < 0.5, bound=rng.random() < 0.5)


# --------------------------------------------------------------------------
# Inputs, drawn on the GPU: the shapes of paper_1310_1854_amd/workloads.py
# --------------------------------------------------------------------------

def _rand(gen, *shape):
    return torch.rand(*shape, dtype=F64, device=DEV, generator=gen)


def _randn(gen, *shape):
    return torch.randn(*shape, dtype=F64, device=DEV, generator=gen)


def _dirs(gen, n):
    z = 2.0 * _rand(gen, n) - 1.0
    phi = 2.0 * math.pi * _rand(gen, n)
    s = torch.sqrt(torch.clamp(1.0 - z * z, min=0.0))
    d = torch.stack([s * torch.cos(phi), s * torch.sin(phi), z], dim=1)
    return d / torch.linalg.vector_norm(d, dim=1, keepdim=True)


def _in_box(gen, n, box):
    lo = torch.tensor(box[:3], dtype=F64, device=DEV)
    hi = torch.tensor(box[3:], dtype=F64, device=DEV)
    return lo + _rand(gen, n, 3) * (hi - lo)


def _inside(p, box):
    lo = torch.tensor(box[:3], dtype=F64, device=DEV)
    hi = torch.tensor(box[3:], dtype=F64, device=DEV)
    return p[((p >= lo) & (p <= hi)).all(dim=1)]


def _until(n, draw_some, box):
    """n points inside the box from a generator of batches (rejection)."""
    got = _inside(draw_some(int(1.1 * n) + 64), box)
    while got.shape[0] < n:
        got = torch.cat([got, _inside(draw_some(int(0.5 * n) + 64), box)])
    return got[:n].contiguous()


def _clumps(gen):
    n = 2000
    sig = 2.0 * torch.exp(math.log(0.01) + (math.log(0.05) - math.log(0.01)) * _rand(gen, n))
    mass = torch.exp(math.log(100.0) * _rand(gen, n))
    cen = -1.0 + 2.0 * sig[:, None] + _rand(gen, n, 3) * (2.0 - 4.0 * sig[:, None])
    return cen, sig, mass


def _from_clumps(gen, clumps, box):
    cen, sig, mass = clumps
    cdf = torch.cumsum(mass, 0) / mass.sum()

    def some(n):
        c = torch.clamp(torch.searchsorted(cdf, _rand(gen, n)), max=cen.shape[0] - 1)
        return cen[c] + _randn(gen, n, 3) * sig[c][:, None]

    return some


def _medium(shape, M, gen):
    """box, sites (M, 3), density (M,), and what ray origins are drawn from."""
    clumps = None
    if shape == "cube":
        box = [-1.0] * 3 + [1.0] * 3
        sites = _in_box(gen, M, box)
        density = _rand(gen, M)
    elif shape == "exp_disc":
        box = [-10.0, -10.0, -3.0, 10.0, 10.0, 3.0]

        def some(n):
            R = -2.5 * torch.log((1.0 - _rand(gen, n)) * (1.0 - _rand(gen, n)))      # Gamma(2, 2.5)
            phi = 2.0 * math.pi * _rand(gen, n)
            u = 2.0 * _rand(gen, n) - 1.0
            z = -0.3 * torch.sign(u) * torch.log1p(-torch.abs(u))                    # Laplace(0.3)
            return torch.stack([R * torch.cos(phi), R * torch.sin(phi), z], dim=1)

        sites = _until(M, some, box)
        density = torch.exp(-torch.hypot(sites[:, 0], sites[:, 1]) / 2.5 - sites[:, 2].abs() / 0.3)
    elif shape == "flared_disc":
        box = [-1000.0] * 3 + [1000.0] * 3

        def height(R):
            return 0.125 * 500.0 * (R / 500.0) ** 1.125

        def some(n):
            R = (1.0 + _rand(gen, n) * (1000.0 ** 2.125 - 1.0)) ** (1.0 / 2.125)
            phi = 2.0 * math.pi * _rand(gen, n)
            z = _randn(gen, n) * height(R) * math.sqrt(2.0 / math.pi)
            return torch.stack([R * torch.cos(phi), R * torch.sin(phi), z], dim=1)

        n_uni = M // 100
        sites = torch.cat([_until(M - n_uni, some, box), _in_box(gen, n_uni, box)])
        R = torch.hypot(sites[:, 0], sites[:, 1]).clamp(min=1e-300)
        rho = (R / 500.0) ** -1.0 * torch.exp(-(math.pi / 4.0) * (sites[:, 2] / height(R)) ** 2)
        density = torch.where((R >= 1.0) & (R <= 1000.0), rho, torch.zeros_like(rho))
    else:
        box = [-1.0] * 3 + [1.0] * 3
        clumps = _clumps(gen)

        def background(n):
            r = -0.5 * torch.log(torch.prod(1.0 - _rand(gen, n, 3), dim=1))          # Gamma(3, 0.5)
            return _dirs(gen, n) * r[:, None]

        sites = torch.cat([_until(M // 2, _from_clumps(gen, clumps, box), box), _until(M - M // 2, background, box)])
        density = torch.exp(-2.0 * torch.linalg.vector_norm(sites, dim=1))
        density[: M // 2] += 1.0
    return box, sites.contiguous(), density.contiguous(), clumps


def _rays(shape, N, box, sites, clumps, gen):
    M = sites.shape[0]
    if shape == "cube":
        return _in_box(gen, N, box), _dirs(gen, N)
    if shape == "clumpy":                                    # half inside clumps, half inward from the faces
        n_in = N // 2
        o_in = _until(n_in, _from_clumps(gen, clumps, box), box)
        n = N - n_in
        o_f = _in_box(gen, n, box)
        d_f = _dirs(gen, n)
        face = torch.randint(0, 6, (n,), device=DEV, generator=gen)
        row, ax = torch.arange(n, device=DEV), face // 2
        sgn = torch.where(face % 2 == 0, -1.0, 1.0).to(F64)
        o_f[row, ax] = sgn
        d_f[row, ax] = -sgn * d_f[row, ax].abs()
        return torch.cat([o_in, o_f]), torch.cat([_dirs(gen, n_in), d_f])
    o = sites[torch.randint(0, M, (N,), device=DEV, generator=gen)]
    if shape == "flared_disc":                               # half from the central source
        o[: N // 2] = 0.0
    return o.contiguous(), _dirs(gen, N)


def _generator(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1_000_003 * int(seed) + salt)


def _medium_and_rays(case, seed):
    gen = _generator(seed, 1)
    box, sites, density, clumps = _medium(case["shape"], case["M"], gen)
    origins, dirs = _rays(case["shape"], case["N"], box, sites, clumps, gen)
    return box, sites, density, origins.contiguous(), dirs.contiguous(), gen


def _spill(n_seg, stride):
    """Spill chunks that paths of these segment counts need past their windows."""
    return int(torch.clamp((n_seg - stride + vrt.SPILL_CHUNK - 1) // vrt.SPILL_CHUNK, min=0).sum())


def _capacity(M, N):
    """Segments that the compact rows of N paths through M cells are given room for."""
    return int(N * (6 + 1.4 * PER_RAY * M ** (1.0 / 3.0)) + 40 * math.sqrt(N) * M ** (1.0 / 3.0))


def _window(M):
    """A window that holds every path of random rays through M cells of the shapes above, a multiple of 16."""
    return int(16 * math.ceil((24.0 + 5.0 * PER_RAY * M ** (1.0 / 3.0)) / 16.0))


def _serve_parts(case):
    shapes = [("cube", 10_000), ("exp_disc", 100_000), ("flared_disc", 1_000_000)]
    grids = [(s, max(1_000, int(m * case["scale"]))) for s, m in shapes]
    lo, hi, n = case["lo"], case["hi"], 12
    sizes = [int(round(lo * (hi / lo) ** (i / (n - 1)))) for i in range(n)]
    reqs = [(i % 3, sizes[(5 * i) % n], "mixed" if (i // 3) % 2 else "fp64") for i in range(n)]
    return grids, reqs


# --------------------------------------------------------------------------
# The cases
# --------------------------------------------------------------------------

def prepare(case, seed):
    op = case["op"]
    if op == "serve":
        parts, reqs = _serve_parts(case)
        grids, media = [], []
        for i, (shape, M) in enumerate(parts):
            box, sites, density, clumps = _medium(shape, M, _generator(seed, 10 + i))
            g = vrt.build_grid(sites, box)
            g.bind_density(density)
            grids.append(g)
            media.append((shape, box, sites, clumps))
        server = vrt.Server(grids, 1 << 30)
        out = []
        for i, (gi, n, mode) in enumerate(reqs):
            shape, box, sites, clumps = media[gi]
            o, d = _rays("exp_disc" if shape != "cube" else "cube", n, box, sites, clumps, _generator(seed, 100 + i))
            b = vrt.TraceBuffers(n)
            vrt.trace_into(grids[gi], o.contiguous(), d.contiguous(), None, b, mode="mixed", grid_density=True)
            out.append((gi, o.contiguous(), d.contiguous(), mode, _spill(b.n_seg, 32) + 8))
        room = sum(_capacity(parts[gi][1], n) for gi, n, _ in reqs)
        rows = [torch.zeros(room, dtype=t, device=DEV) for t in (torch.int32, F64)]
        torch.cuda.synchronize()
        return dict(case=case, server=server, reqs=out, rows=rows)
    if op == "build":
        box, sites, _, _ = _medium(case["shape"], case["M"], _generator(seed, 1))
        return dict(case=case, box=box, sites=sites, col=torch.zeros(20 * case["M"] + 64, dtype=torch.int32, device=DEV))
    if op == "locate":
        gen = _generator(seed, 1)
        box, sites, _, _ = _medium(case["shape"], case["M"], gen)
        grid = vrt.build_grid(sites, box, block_lists=case["blocks"])
        return dict(case=case, grid=grid, pts=_in_box(gen, case["N"], box))
    box, sites, density, origins, dirs, gen = _medium_and_rays(case, seed)
    grid = vrt.build_grid(sites, box, block_lists=True)
    if case["bound"]:
        grid.bind_density(density)
    s = dict(case=case, grid=grid, o=origins, d=dirs, rho=None if case["bound"] else density)
    N = case["N"]
    if op == "paths":
        b = vrt.TraceBuffers(N, ordered=case["ordered"])
        vrt.trace_into(grid, origins, dirs, None, b, mode="mixed", ordered=case["ordered"], persistent=case["ordered"])
        room = _capacity(case["M"], N)
        if int(b.n_seg.sum(dtype=torch.int64)) > room:
            raise RuntimeError("the rows of this case need more room")
        s["bufs"] = vrt.TraceBuffers(N, seg_stride=STRIDE, spill_chunks=_spill(b.n_seg, STRIDE) + 1,
                                     ordered=case["ordered"])
        s["cell"] = torch.zeros(room, dtype=torch.int32, device=DEV)   # entries past the last row stay as they are here
        s["len"] = torch.zeros(room, dtype=F64, device=DEV)
    elif op == "windows":
        s["bufs"] = vrt.TraceBuffers(N, seg_stride=_window(case["M"]), ordered=case["ordered"])
        s["bufs"].seg_cell.zero_()   # the slots past a path's end stay as they are here
        s["bufs"].seg_len.zero_()
    elif op == "depth":
        s["bufs"] = vrt.TraceBuffers(N, ordered=case["ordered"])
    elif op == "transport":
        mean = float(density.mean()) * (box[3] - box[0])
        s["kappa"] = 2.0 / max(mean, 1e-300)
        s["tau_stop"] = -torch.log(1.0 - _rand(gen, N))
        s["weight"] = 0.5 + _rand(gen, N)
    return s


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "build":
        grid = vrt.build_grid(s["sites"], s["box"], block_lists=c["blocks"])
        row_ptr, col = grid.neighbors()
        s["col"][: col.numel()].copy_(col)   # into the program's own table
        out = dict(row_ptr=row_ptr, col=s["col"], volume=grid.volumes())
        if c["blocks"]:
            out["bbox"] = grid.bboxes()
        grid.free()
        return out
    if op == "locate":
        return dict(cell=(vrt.locate_blocks if c["blocks"] else vrt.locate)(s["grid"], s["pts"]))
    if op == "serve":
        srv = s["server"]
        ids = [srv.submit(gi, o, d, None, mode=mode, seg_stride=32, spill_chunks=chunks, grid_density=True)
               for gi, o, d, mode, chunks in s["reqs"]]
        out = []
        for rid in ids:
            srv.wait(rid)
            r = srv.result(rid)
            srv.release(rid)
            out.append(r)
        cells, lens = [r["seg_cell"] for r in out], [r["seg_len"] for r in out]
        total = sum(x.numel() for x in cells)
        torch.cat(cells, out=s["rows"][0][:total])   # into the program's own rows
        torch.cat(lens, out=s["rows"][1][:total])
        return dict(rows=s["rows"], per_request=[[r["tau"], r["n_seg"], r["ray_off"]] for r in out])
    kw = dict(mode=c["mode"], ordered=c["ordered"], persistent=c["ordered"], grid_density=c["bound"])
    if op == "transport":
        r = vrt.trace(s["grid"], s["o"], s["d"], s["rho"], kappa=s["kappa"], segments="none", tallies=True,
                      tau_stop=s["tau_stop"], weight=s["weight"], **kw)
        return {k: r[k] for k in ("tau", "n_seg", "status", "stop_cell", "stop_s", "tally_len", "tally_abs")}
    b = s["bufs"]
    vrt.trace_into(s["grid"], s["o"], s["d"], s["rho"], b, **kw)
    out = dict(tau=b.tau, n_seg=b.n_seg, status=b.status)
    if op == "paths":
        off = vrt.exclusive_scan(b.n_seg)
        vrt.gather_paths(b, off, s["cell"], s["len"])
        out.update(ray_off=off, seg_cell=s["cell"], seg_len=s["len"])
    elif op == "windows":
        out.update(seg_cell=b.seg_cell, seg_len=b.seg_len)
    return out


def _trace_work(M, N, segments):
    """Bytes and operations of N paths through M cells: rays and results, the cells that are met (site, density and
    neighbour indices of each once), segments written; one crossing of some 20 operations per neighbour and step."""
    steps = PER_RAY * M ** (1.0 / 3.0) * N
    cells = min(float(M), steps)
    return dict(bytes=N * (48 + 13) + cells * (24 + 8 + 4 * NEIGHBOURS) + (12 * steps if segments else 0),
                flops=steps * NEIGHBOURS * 20)


def work(case):
    op = case["op"]
    if op == "serve":
        parts, reqs = _serve_parts(case)
        all_of = [_trace_work(parts[gi][1], n, True) for gi, n, _ in reqs]
        return {k: sum(w[k] for w in all_of) for k in ("bytes", "flops")}
    M = case["M"]
    if op == "build":   # sites in; lists, volumes (and boxes) out; each neighbour's plane against some 27 vertices
        return dict(bytes=M * (24 + 8 + 4 * NEIGHBOURS + 8 + (48 if case["blocks"] else 0)),
                    flops=M * NEIGHBOURS * 27 * 6)
    N = case["N"]
    if op == "locate":
        return dict(bytes=N * 28 + 24 * min(M, 8 * N), flops=N * 8 * 8)
    w = _trace_work(M, N, op in ("paths", "windows"))
    if op == "transport":
        w["bytes"] += 36 * N + 16 * M
    return w


def _brute_paths(sites, box, density, origins, dirs):
    """Whole paths by testing every site at every step: lists of segment lengths and the optical depth of each ray."""
    N, M = origins.shape[0], sites.shape[0]
    k = dirs / torch.linalg.vector_norm(dirs, dim=1, keepdim=True)
    lo, hi = (torch.tensor(v, dtype=F64, device=DEV) for v in (box[:3], box[3:]))
    far = torch.where(k > 0, hi, lo)
    L = torch.where(k != 0, (far - origins) / k, torch.full_like(k, math.inf)).min(dim=1).values
    tau = torch.zeros(N, dtype=F64, device=DEV)
    lens, rays = [], []
    step = max(1, int(2e7 // M))
    for a in range(0, N, step):
        idx = torch.arange(a, min(N, a + step), device=DEV)
        o = origins[idx]
        cur = torch.cdist(o, sites, compute_mode="donot_use_mm_for_euclid_dist").argmin(dim=1)
        s = torch.zeros(idx.shape[0], dtype=F64, device=DEV)
        while idx.numel():
            r0, kk, pm = origins[idx], k[idx], sites[cur]
            den = torch.zeros(idx.shape[0], M, dtype=F64, device=DEV)
            num = torch.zeros_like(den)
            for x in range(3):
                n = sites[None, :, x] - pm[:, None, x]
                den += n * kk[:, None, x]
                num += n * (0.5 * (sites[None, :, x] + pm[:, None, x]) - r0[:, None, x])
            t = torch.where(den > 0, num / den, torch.full_like(den, math.inf))
            best, nxt = t.min(dim=1)
            end = best >= L[idx]
            best = torch.where(end, L[idx], best)
            ln = best - s
            emit = ln > 0
            tau[idx] += torch.where(emit, density[cur] * ln, torch.zeros_like(ln))
            lens.append(ln[emit])
            rays.append(idx[emit])
            keep = ~end
            s = torch.maximum(s, best)[keep]
            idx, cur = idx[keep], nxt[keep]
    lens, rays = torch.cat(lens), torch.cat(rays)
    order = torch.argsort(rays, stable=True)
    return tau, lens[order], torch.bincount(rays, minlength=N)


def exact(case, seed):
    op = case["op"]
    if op not in ("paths", "windows", "depth") or case["M"] * case["N"] > 2e7 or case["M"] > 200_000:
        return None     # cells are whole numbers; brute force over the others takes minutes
    box, sites, density, origins, dirs, _ = _medium_and_rays(case, seed)
    tau, lens, count = _brute_paths(sites, box, density, origins, dirs)
    out = dict(tau=tau, n_seg=None, status=None)
    if op == "paths":
        rows = torch.zeros(_capacity(case["M"], case["N"]), dtype=F64, device=DEV)
        rows[: lens.numel()] = lens
        out.update(ray_off=None, seg_cell=None, seg_len=rows)
    elif op == "windows":
        stride = _window(case["M"])
        first = torch.cumsum(count, 0) - count
        ray = torch.repeat_interleave(torch.arange(case["N"], device=DEV), count)
        rows = torch.zeros(case["N"] * stride, dtype=F64, device=DEV)
        rows[ray * stride + torch.arange(lens.numel(), device=DEV) - first[ray]] = lens
        out.update(seg_cell=None, seg_len=rows)
    return out
