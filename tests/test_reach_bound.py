"""Where an exit search may stop, checked numerically on the CPU.

Rows list their neighbours nearest first, and a search ends at a neighbour at
squared distance n2 from the cell's site when n2 / 4 > 1.0003 rho^2 + reach,
rho being the larger of the distances of the current point and of the best
crossing (or its upper bound) from the site: the bisector then lies beyond both
ends of the way between them. The claim is that no such neighbour has an FP64
crossing, as the FP64 step computes it, at or before the best one. It is
checked on planes at and just past that line, which the rule is least sure of:
square on to either end, random, nearly parallel to the ray (down to a rounding
of n.k), with the best crossing ahead and behind, origins far along the ray and
boxes far from the origin of the coordinates; for the FP64 search, the one over
FP32 records and the one over compact records.
"""
import numpy as np
import pytest

from tests.test_mixed_bound import F, Q_SHIFT, cross64, fma

N = 400_000


def _case(rng, kind, far):
    scale = 10.0 ** rng.uniform(-4, 1, N)
    pm = far + rng.uniform(-100, 100, (N, 3))
    k = rng.normal(size=(N, 3))
    k /= np.linalg.norm(k, axis=1, keepdims=True)
    q = pm + rng.normal(size=(N, 3)) * (scale * rng.uniform(0, 1, N))[:, None]
    s_c = np.where(rng.random(N) < 0.3, 0.0, 10.0 ** rng.uniform(-3, 2.2, N))
    r0 = q - s_c[:, None] * k
    t = scale * rng.uniform(-0.2, 2.0, N)                      # the best crossing from the current point
    cur, x = (r0 + s_c[:, None] * k) - pm, (r0 + (s_c + t)[:, None] * k) - pm
    rho = np.sqrt(np.maximum((cur * cur).sum(1), (x * x).sum(1)))
    if kind == "ends":
        d = np.where(rng.random((N, 1)) < 0.5, x, cur)
    elif kind == "graze":
        d = rng.normal(size=(N, 3))
        d -= (d * k).sum(1, keepdims=True) * k
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        d += k * 10.0 ** rng.uniform(-17, -2, (N, 1))
    else:
        d = rng.normal(size=(N, 3))
    d /= np.maximum(np.linalg.norm(d, axis=1, keepdims=True), 1e-300)
    pj = pm + d * (2 * rho * np.sqrt(1.0003) * (1 + 10.0 ** rng.uniform(-9, -1, N) * rng.choice([-0.1, 1, 1], N)))[:, None]
    pts = np.abs(np.stack([pm, pj, r0], axis=1))
    diag = np.linalg.norm(np.ptp(np.stack([pm, pj, r0], axis=1), axis=1), axis=1)
    eps_abs = (2.0 ** -48 * (2 * pts.max(axis=(1, 2)) + diag)).astype(F)
    return pm, pj, r0, k, s_c, t, eps_abs, cur, x, scale


def _check(stop, pm, pj, r0, k, s_best):
    assert stop.sum() > N // 20                                 # the line is met from both sides
    with np.errstate(divide="ignore", invalid="ignore"):
        s, den = cross64(pj, pm, r0, k)
    bad = stop & (den > 0) & ~(s > s_best)
    assert not bad.any(), (int(bad.sum()), np.flatnonzero(bad)[:3])


def _rho2_32(q, k32, t32):
    x = fma(t32, k32[:, 0], q[:, 0]), fma(t32, k32[:, 1], q[:, 1]), fma(t32, k32[:, 2], q[:, 2])
    qq = (q[:, 0] * q[:, 0] + q[:, 1] * q[:, 1]) + q[:, 2] * q[:, 2]
    return np.maximum(qq, fma(x[0], x[0], fma(x[1], x[1], (x[2] * x[2]).astype(F))))


@pytest.mark.parametrize("far", [0.0, 1e6])
@pytest.mark.parametrize("kind", ["ends", "graze", "random"])
def test_fp64_search(kind, far):
    pm, pj, r0, k, s_c, t, e, cur, x, _ = _case(np.random.default_rng(len(kind)), kind, far)
    n = pj - pm
    nn = (n[:, 0] * n[:, 0] + n[:, 1] * n[:, 1]) + n[:, 2] * n[:, 2]
    rho2 = np.maximum((cur[:, 0] ** 2 + cur[:, 1] ** 2) + cur[:, 2] ** 2, (x[:, 0] ** 2 + x[:, 1] ** 2) + x[:, 2] ** 2)
    reach = 4e5 * e.astype(np.float64) ** 2
    _check(0.25 * nn > 1.0003 * rho2 + reach, pm, pj, r0, k, s_c + t)


@pytest.mark.parametrize("far", [0.0, 1e6])
@pytest.mark.parametrize("kind", ["ends", "graze", "random"])
def test_fp32_records(kind, far):
    pm, pj, r0, k, s_c, t, e, cur, _, _ = _case(np.random.default_rng(10 + len(kind)), kind, far)
    n, t32 = (pj - pm).astype(F), t.astype(F)
    reach = np.clip(4e5 * e.astype(np.float64) ** 2, 1e-36, 3e38).astype(F)
    n2 = fma(n[:, 0], n[:, 0], fma(n[:, 1], n[:, 1], (n[:, 2] * n[:, 2]).astype(F)))
    stop = F(0.25) * n2 > fma(F(1.0003), _rho2_32(cur.astype(F), k.astype(F), t32), reach)
    _check(stop, pm, pj, r0, k, s_c + t32.astype(np.float64))


@pytest.mark.parametrize("far", [0.0, 1e6])
@pytest.mark.parametrize("kind", ["ends", "graze", "random"])
def test_compact_records(kind, far):
    rng = np.random.default_rng(20 + len(kind))
    pm, pj, r0, k, s_c, t, e, cur, _, _ = _case(rng, kind, far)
    n = pj - pm
    E = np.frexp(np.abs(n).max(axis=1))[1] + rng.integers(0, 9, N)      # the row's largest offset may be larger
    qs = np.ldexp(1.0, Q_SHIFT - E)
    i = np.abs(np.rint(n * qs[:, None]))
    assert i.max() <= 2 ** 19
    e_s = (e.astype(np.float64) * qs).astype(F)
    reach = fma((F(4e5) * e_s).astype(F), e_s, F(1.0))
    last = np.maximum(i.astype(F) - F(1.0), F(0.0))
    n2 = fma(last[:, 0], last[:, 0], fma(last[:, 1], last[:, 1], (last[:, 2] * last[:, 2]).astype(F)))
    t32 = (t * qs).astype(F)
    stop = F(0.25) * n2 > fma(F(1.0003), _rho2_32((cur * qs[:, None]).astype(F), k.astype(F), t32), reach)
    _check(stop, pm, pj, r0, k, s_c + t32.astype(np.float64) / qs)
