"""The pair filters of the encounter checks keep every pair that can be flagged.

First the claim on the Hermite data: with chord midpoints M, chords c, half
differences d = dt (V0 - V1)/2 and means p = dt (V0 + V1)/2 - c of the endpoint
velocity deviations, a pair with D > C + 3/4 (|d_j - d_i| + 0.385 (|p_i| + |p_j|)) +
rc_ij (D, C the distances of the midpoints and chords) stays outside rc_ij, against the
oracle's exact minimum on arbitrary data and on Kepler arcs.

Then the matrix-core filter of the direct check: emulation of its records (M and c as
two FP16 values, d' and s' as one, the body's share of the error bound taken off)
against the condition D <= C + 3/4 |d_j - d_i| + s_i + s_j, pairs placed at the
boundary and just inside, with the summation error of the product at its measured
worst (2^-21 of the terms' magnitudes)."""
import numpy as np
import pytest

import oracle
import workloads

P = 0.385                                            # kEncP
K1, K2, K3 = 2.0 ** -17, 2.0 ** -20, 2.0 ** -28      # enc_record's shares
MAX, UNIT, OUT = 8.0, 64.0, -60000.0
R98, R2 = np.sqrt(9.0 / 8.0), np.sqrt(2.0)


# ------------------------------------------------------------------ the claim

def geometry(dt, q0, v0, q1, v1):
    c = q1 - q0
    d = 0.5 * dt * (v0 - v1)
    p = P * np.linalg.norm(0.5 * dt * (v0 + v1) - c)
    return 0.5 * (q0 + q1), c, d, p


def reach(gi, gj, rcij):
    C = np.linalg.norm(gj[1] - gi[1])
    return C + 0.75 * (np.linalg.norm(gj[2] - gi[2]) + gi[3] + gj[3]) + rcij


def _body(rng, scale):
    q0 = rng.normal(size=3) * scale
    q1 = q0 + rng.normal(size=3) * scale * rng.uniform(0, 2)
    return q0, rng.normal(size=3), q1, rng.normal(size=3) * rng.uniform(0, 3)


def test_pairs_outside_the_reach_stay_outside_rc():
    rng = np.random.default_rng(2025)
    for trial in range(20000):
        dt = rng.uniform(0.01, 2.0) * rng.choice([-1, 1])
        bi = _body(rng, rng.uniform(0.01, 1))
        if trial % 2:                    # a neighbour: nearly the same motion
            e = rng.uniform(0, 0.1)
            bj = [t + e * rng.normal(size=3) for t in bi]
        else:
            bj = list(_body(rng, rng.uniform(0.01, 1)))
        rc = rng.uniform(0, 0.5, 2) * rng.choice([1e-3, 1.0])
        gi, gj = geometry(dt, *bi), geometry(dt, *bj)
        u = rng.normal(size=3)
        u /= np.linalg.norm(u)
        shift = gi[0] + u * reach(gi, gj, rc.max()) * (1 + rng.uniform(1e-9, 0.05)) - gj[0]
        bj[0], bj[2] = bj[0] + shift, bj[2] + shift
        d2 = oracle.pair_min_d2(dt, *bi, *bj)
        assert d2 > rc.max() ** 2, (trial, d2, rc)


def test_flagged_pairs_of_a_dense_ring_are_within_the_reach():
    w = workloads.ring(400, m=1e-7)
    Q0, V0 = oracle.helio_to_dh(1.0, w.m, w.x, w.v)
    rc = oracle.rcrit(1.0, w.m, Q0)
    for dt in (0.04, 0.2):
        Q1, V1, _ = oracle.drift(w.G * 1.0, dt, Q0, V0)
        e = oracle.encounters(dt, Q0, V0, Q1, V1, rc)
        g = [geometry(dt, Q0[i], V0[i], Q1[i], V1[i]) for i in range(400)]
        flagged = list(zip(e["ice"].tolist(), e["jce"].tolist()))
        assert len(flagged) > 5
        near = 0
        for i in range(400):
            for j in range(i + 1, 400):
                near += np.linalg.norm(g[j][0] - g[i][0]) <= reach(g[i], g[j], max(rc[i], rc[j]))
        for i, j in flagged:
            assert np.linalg.norm(g[j][0] - g[i][0]) <= reach(g[i], g[j], max(rc[i], rc[j]))
        assert dt > 0.1 or near < 400 * 399 // 8     # and it does cull


# ------------------------------------------------------------------ the records

def record(M, c, d, s, inv_l):
    u = np.concatenate([M, c], axis=1) * inv_l
    hi = u.astype(np.float16).astype(np.float64)
    lo = (u - hi).astype(np.float16).astype(np.float64)
    w = R98 * inv_l * d
    D = w.astype(np.float16).astype(np.float64)
    sp = R2 * (s * inv_l) + 2.0 ** -11 * np.sqrt(np.sum(w ** 2, axis=1)) + 2.0 ** -23
    sh = (sp * (1.0 + 2.0 ** -10)).astype(np.float16).astype(np.float64)
    m2 = np.sum(u[:, :3] ** 2, axis=1)
    c2 = 2.0 * (np.sum(u[:, 3:] ** 2, axis=1) + np.sum(D ** 2, axis=1) + sh ** 2)
    nn = m2 + c2
    al = (m2 - c2 - (K1 * nn + K2 * np.sqrt(nn) + K3)) * UNIT
    inside = np.all(np.abs(u) <= MAX, axis=1) & np.all(np.abs(w) <= MAX, axis=1) & (sp <= 0.5 * MAX)
    keep = inside[:, None]
    al = np.where(inside, al, OUT)
    ah = al.astype(np.float16).astype(np.float64)
    alo = np.where(inside, (al - ah).astype(np.float16).astype(np.float64), 0.0)
    return np.where(keep, hi, 0.0), np.where(keep, lo, 0.0), np.where(keep, D, 0.0), \
        np.where(inside, sh, 0.0), ah, alo


def phi(ri, rj, pessimistic):
    """The filter's value (candidate: below zero), pushed up by the worst summation error."""
    g = np.array([-2.0, -2.0, -2.0, 4.0, 4.0, 4.0])
    hi, li, di, si, ai, bi = ri
    hj, lj, dj, sj, aj, bj = rj
    terms = [g * hi * hj, g * li * hj, g * hi * lj, 4.0 * di * dj, (-4.0 * si * sj)[:, None]]
    al_i = np.float32((np.float32(ai) + np.float32(bi)) * np.float32(1.0 / UNIT)).astype(np.float64)
    rest = [aj / UNIT, bj / UNIT, al_i]
    val = sum(np.sum(t, axis=1) for t in terms) + sum(rest)
    mag = sum(np.sum(np.abs(t), axis=1) for t in terms) + sum(np.abs(t) for t in rest)
    return val + (2.0 ** -21 * mag if pessimistic else 0.0)


def pairs(rng, n, lo, hi, scale_c, scale_d, scale_s):
    """Bodies i anywhere in the shell [lo, hi], bodies j at `t` times the boundary distance."""
    def unit():
        d = rng.normal(size=(n, 3))
        return d / np.linalg.norm(d, axis=1)[:, None]
    Mi = unit() * (10.0 ** rng.uniform(np.log10(lo), np.log10(hi), n))[:, None]
    ci = rng.normal(size=(n, 3)) * scale_c
    cj = ci + rng.normal(size=(n, 3)) * scale_c * (10.0 ** rng.uniform(-4, 0, n))[:, None]
    di = rng.normal(size=(n, 3)) * scale_d
    dj = di + rng.normal(size=(n, 3)) * scale_d * (10.0 ** rng.uniform(-4, 0, n))[:, None]
    s = 10.0 ** rng.uniform(-8, np.log10(scale_s), (2, n))
    bound = np.linalg.norm(cj - ci, axis=1) + 0.75 * np.linalg.norm(dj - di, axis=1) + s[0] + s[1]
    t = np.where(rng.random(n) < 0.5, 1.0, rng.uniform(0.99, 1.0, n))
    Mj = Mi + unit() * (bound * t)[:, None]
    return (Mi, ci, di, s[0]), (Mj, cj, dj, s[1])


@pytest.mark.parametrize("lo,hi,scale_c,scale_d,scale_s", [
    (1.0, 3.0, 0.3, 0.02, 0.02), (0.5, 5.0, 0.01, 1e-4, 0.005), (0.9, 1.1, 0.25, 0.03, 5e-4),
    (1e-3, 7.9, 0.5, 0.3, 1e-3), (0.01, 0.02, 1e-3, 1e-5, 1e-5), (0.9, 1.1, 1.5, 1.0, 0.5)])
def test_no_flaggable_pair_is_dropped(lo, hi, scale_c, scale_d, scale_s):
    rng = np.random.default_rng(11)
    i, j = pairs(rng, 40000, lo, hi, scale_c, scale_d, scale_s)
    for unit in (1.0, 0.5, 2.0 ** -3):          # 1/L: the system's largest distance and larger units
        p = phi(record(*i, unit), record(*j, unit), True)
        assert np.all(p < 0.0), (unit, p.max())


def test_body_outside_the_unit_is_always_a_candidate():
    rng = np.random.default_rng(12)
    i, j = pairs(rng, 2000, 1.0, 8.0, 0.3, 0.02, 0.02)
    far = (i[0] * 100.0, i[1], i[2], i[3])
    wide = (i[0], i[1], i[2], i[3] + 10.0)
    for o in (far, wide):
        assert np.all(phi(record(*o, 1.0), record(*j, 1.0), True) < 0.0)
        assert np.all(phi(record(*o, 1.0), record(*o, 1.0), True) < 0.0)


def test_distant_pairs_are_dropped():
    rng = np.random.default_rng(13)
    i, j = pairs(rng, 20000, 1.0, 3.0, 0.05, 0.01, 0.005)
    # 0.3 length units beyond the boundary
    e = j[0] - i[0]
    e /= np.linalg.norm(e, axis=1)[:, None]
    out = (j[0] + 0.3 * e, j[1], j[2], j[3])
    assert np.all(phi(record(*i, 0.25), record(*out, 0.25), False) > 0.0)


def test_sorted_filter_keeps_flaggable_pairs():
    """The FP32 form of the sorted check, with the widening of its records."""
    F = np.float32
    rng = np.random.default_rng(14)
    for lo, hi, sc, sd, ss in ((0.9, 1.1, 0.25, 0.03, 5e-4), (0.5, 50.0, 0.01, 1e-4, 5e-3), (1.0, 3.0, 1.0, 0.5, 0.1)):
        i, j = pairs(rng, 40000, lo, hi, sc, sd, ss)

        def rec(M, c, d, s):
            w = (s + 2.0 ** -21 * sum(np.abs(t).sum(axis=1) for t in (M, c, d))) * (1.0 + 2.0 ** -18)
            return M.astype(F), c.astype(F), d.astype(F), w.astype(F)
        a, b = rec(*i), rec(*j)
        sq = [np.sum((b[k] - a[k]) ** 2, axis=1, dtype=F) for k in range(3)]
        S = a[3] + b[3]
        rhs = (F(2.0) * S * S + (F(1.125) * sq[2] + sq[1])) * F(2.0 * (1.0 + 2.0 ** -18))
        assert np.all(sq[0] <= rhs)
