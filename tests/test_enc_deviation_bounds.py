"""What the encounter filters conclude from the endpoint velocity deviations: half the
difference d = dt (V0 - V1)/2 and the mean p = dt (V0 + V1)/2 - c, with E = |d_j - d_i| +
0.385 (|p_i| + |p_j|), D and C the distances of the chord midpoints and chords, a = C/2.

  (A) D > C + 3/4 E + rc leaves the pair outside rc;
  (B) where D > a and g = (D - a)^2 - (D + a) E/2 > 0, the squared distance stays >= g,
      from which come the cull of tile pairs and the test of one body against a tile.

The squared distance is the cubic with slopes 2 dt dQ0.dV0 and 2 dt dQ1.dV1, so that p
acts along the chord too: the data here have |p| up to hundreds of chords, along and
against the chord.  The tile bounds are those of the sorted check (centre and radius of
M, c and d, the radius of d with 0.385 |p| in it), one body against a tile from its FP32
records."""
import numpy as np
import pytest

import oracle

P = 0.385


def minimum(f0, f1, g0, g1):
    """The least value over [0, 1] of the cubic with these ends and slopes."""
    b, c = 3 * (f1 - f0) - 2 * g0 - g1, 2 * (f0 - f1) + g0 + g1
    f = lambda s: f0 + s * (g0 + s * (b + s * c))  # noqa: E731
    best = np.minimum(f0, f1)
    with np.errstate(divide="ignore", invalid="ignore"):
        q = -0.5 * (2 * b + np.copysign(np.sqrt(4 * b * b - 12 * c * g0), b))
        for s in (q / (3 * c), g0 / q, -g0 / (2 * b)):
            best = np.where((s > 0) & (s < 1), np.minimum(best, f(np.nan_to_num(s))), best)
    return best


def relative(rng, n):
    """Relative c, d, p of n pairs: each of them long or short beside the others, p often
    along or against c, d often along or against both."""
    def unit():
        u = rng.normal(size=(n, 3))
        return u / np.linalg.norm(u, axis=1)[:, None]
    c = unit() * (10.0 ** rng.uniform(-2, 0.3, n))[:, None]
    e = c / np.linalg.norm(c, axis=1)[:, None]
    mix = lambda: np.where((rng.random(n) < 0.5)[:, None], e * rng.choice([-1, 1], n)[:, None], unit())  # noqa: E731
    d = mix() * (10.0 ** rng.uniform(-4, 2.5, n))[:, None]
    p = mix() * (10.0 ** rng.uniform(-4, 2.5, n))[:, None]
    return c, d, p, mix()


def cubic(M, c, d, p):
    q0, q1 = M - 0.5 * c, M + 0.5 * c
    f0, f1 = np.sum(q0 * q0, 1), np.sum(q1 * q1, 1)
    return minimum(f0, f1, 2 * np.sum(q0 * (c + p + d), 1), 2 * np.sum(q1 * (c + p - d), 1))


def norm(x):
    return np.linalg.norm(x, axis=1)


@pytest.mark.parametrize("seed", range(2))
def test_outside_the_reach(seed):
    rng = np.random.default_rng(100 + seed)
    c, d, p, u = relative(rng, 200000)
    rc = np.where(rng.random(len(c)) < 0.3, 0.0, 10.0 ** rng.uniform(-4, 1, len(c)))
    D = (norm(c) + 0.75 * (norm(d) + P * norm(p)) + rc) * (1 + 10.0 ** rng.uniform(-9, -1, len(c)))
    low = cubic(u * D[:, None], c, d, p)
    assert np.all(low > rc * rc * (1 - 1e-9))


@pytest.mark.parametrize("seed", range(2))
def test_bound_where_positive(seed):
    rng = np.random.default_rng(200 + seed)
    c, d, p, u = relative(rng, 200000)
    a, E = 0.5 * norm(c), norm(d) + P * norm(p)
    # D from just above where g turns positive: (D - a)^2 = (D + a) E / 2
    root = a + 0.25 * E + np.sqrt(E * E / 16 + a * E)
    D = root * (1 + 10.0 ** rng.uniform(-8, 1, len(c)))
    g = (D - a) ** 2 - 0.5 * (D + a) * E
    low = cubic(u * D[:, None], c, d, p)
    assert np.all(g > 0) and np.all(low >= g - 1e-12 * (D + a) ** 2)


def test_factors_of_the_argument():
    """The two inequalities in t = |1 - 2s| (and x = D/a) on which (A) and (B) rest."""
    t = np.linspace(0.0, 1.0, 20001)
    al, be = 0.5 * (1 - t * t), 0.5 * t * (1 - t * t)
    assert be.max() < P / 2
    assert np.min((2 - t) * (1.5 * P - be) - al * (1 + t * t)) > 0.1
    x = 1.0 + np.concatenate([[0.0], 10.0 ** np.linspace(-8, 8, 1601)])[:, None]
    t = t[::20]
    lhs, rhs = (1 - t) * (2 * x - 1 - t) * (x + 1), ((1 - t * t) / P - 1) * (x - 1) ** 2
    assert np.all(lhs - rhs >= -1e-12 * x * x)
    assert np.all(2 * (1 - t) - ((1 - t * t) / P - 1) > 0)         # the leading terms for x -> infinity


# ------------------------------------------------------------------ tiles

def geometry(b, dt):
    q0, v0, q1, v1 = b
    c = q1 - q0
    return 0.5 * (q0 + q1), c, 0.5 * dt * (v0 - v1), P * np.linalg.norm(0.5 * dt * (v0 + v1) - c)


def tile_bounds(bodies, rcs, dt):
    g = [geometry(b, dt) for b in bodies]
    M, C, d = (np.array([t[k] for t in g]) for k in range(3))
    p = np.array([t[3] for t in g])
    cm, cc, ce = M.mean(0), C.mean(0), d.mean(0)
    w = 1 + 2.0 ** -20
    return (cm, w * np.max(norm(M - cm)), cc, w * np.max(norm(C - cc)), ce, w * np.max(norm(d - ce) + p), max(rcs))


def lane_ball(body, rc, dt):
    f = np.float32
    M, c, d, p = geometry(body, dt)
    M, c, d = (x.astype(f).astype(np.float64) for x in (M, c, d))
    n = np.linalg.norm
    return (M, 2.0 ** -23 * n(M), c, 2.0 ** -23 * n(c), d, float(f(p * (1 + 2.0 ** -20))) + 2.0 ** -23 * n(d),
            float(f(rc * (1 + 2.0 ** -20))))


def may_meet(A, B):
    n = np.linalg.norm
    D = n(B[0] - A[0])
    Cm = n(B[2] - A[2]) + A[3] + B[3]
    Em = n(B[4] - A[4]) + A[5] + B[5]
    Lmin, Qmax = D - A[1] - B[1] - 0.5 * Cm, D + A[1] + B[1] + 0.5 * Cm
    RC = max(A[6], B[6])
    return not (Lmin > 0 and Lmin * Lmin - 0.5 * Qmax * Em > RC * RC * (1 + 1e-6) + 1e-12 * Qmax * Qmax)


def tile(rng, k, spread, dt, dominant):
    """k bodies whose midpoints, chords and deviations cluster; `dominant`: the mean
    deviations are the largest of these and lie along the chords."""
    q = rng.normal(size=3)
    c = rng.normal(size=3) * spread * rng.uniform(0.5, 5)
    d = rng.normal(size=3) * spread * rng.uniform(0, 2)
    p = c * rng.uniform(-6, 6) if dominant else rng.normal(size=3) * spread * 0.2
    out = []
    for _ in range(k):
        q0 = q + rng.normal(size=3) * spread
        ci = c + rng.normal(size=3) * spread * 0.3
        di, pi = d + rng.normal(size=3) * spread * 0.1, p + rng.normal(size=3) * spread * 0.1
        out.append((q0, (ci + pi + di) / dt, q0 + ci, (ci + pi - di) / dt))
    return out


def moved(bodies, shift):
    return [(b[0] + shift, b[1], b[2] + shift, b[3]) for b in bodies]


def centre(bodies):
    return np.mean([0.5 * (b[0] + b[2]) for b in bodies], 0)


def at_the_edge(rng, A, B, bounds_a, bounds_b):
    """B moved along the line of the centres: to just about the distance at which the two
    bounds stop meeting, or anywhere closer (where pairs are flagged)."""
    u = centre(B) - centre(A)
    u /= np.linalg.norm(u)
    meet = lambda r: may_meet(bounds_a(A), bounds_b(moved(B, centre(A) + u * r - centre(B))))  # noqa: E731
    hi = 1e-6
    while meet(hi):
        hi *= 2
    lo = hi / 2
    for _ in range(12):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if meet(mid) else (lo, mid)
    return moved(B, centre(A) + u * hi * rng.uniform(*((0.9, 1.05) if rng.random() < 0.4 else (0.0, 0.9))) - centre(B))


@pytest.mark.parametrize("dominant", [False, True])
def test_tile_pairs(dominant):
    rng = np.random.default_rng(77)
    culled = flagged = 0
    for trial in range(120):
        dt = rng.uniform(0.01, 0.2)
        spread = 10 ** rng.uniform(-3, -1)
        A, B = tile(rng, 6, spread, dt, dominant), tile(rng, 6, spread, dt, dominant)
        ra, rb = rng.uniform(0, 3 * spread, 6), rng.uniform(0, 3 * spread, 6)
        ba, bb = (lambda t: tile_bounds(t, ra, dt)), (lambda t: tile_bounds(t, rb, dt))
        B = at_the_edge(rng, A, B, ba, bb)
        ok = may_meet(ba(A), bb(B))
        culled += not ok
        for i, x in enumerate(A):
            for j, y in enumerate(B):
                if oracle.pair_min_d2(dt, *x, *y) <= max(ra[i], rb[j]) ** 2:
                    flagged += 1
                    assert ok, trial
    assert culled > 8 and flagged > 20


@pytest.mark.parametrize("dominant", [False, True])
def test_one_body_against_a_tile(dominant):
    rng = np.random.default_rng(99)
    culled = flagged = 0
    for trial in range(240):
        dt = rng.uniform(0.01, 0.2)
        spread = 10 ** rng.uniform(-3, -1)
        A, B = tile(rng, 1, spread, dt, dominant), tile(rng, 8, spread, dt, dominant)
        ra, rb = rng.uniform(0, 3 * spread), rng.uniform(0, 3 * spread, 8)
        ba, bb = (lambda t: lane_ball(t[0], ra, dt)), (lambda t: tile_bounds(t, rb, dt))
        B = at_the_edge(rng, A, B, ba, bb)
        ok = may_meet(ba(A), bb(B))
        culled += not ok
        for j, y in enumerate(B):
            if oracle.pair_min_d2(dt, *A[0], *y) <= max(ra, rb[j]) ** 2:
                flagged += 1
                assert ok, trial
    assert culled > 16 and flagged > 20
