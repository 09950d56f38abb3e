"""The matrix-core filter of the direct encounter check keeps every pair that can be
flagged: emulation of its records (two FP16 values per component, the body's share
of the error bound taken off) against the FP64 condition
D^2 <= 2 C^2 + 2 (b_i + b_j + max(rc_i, rc_j))^2, pairs placed at the boundary and
just inside, with the summation error of the product at its measured worst
(2^-21 of the terms' magnitudes)."""
import numpy as np
import pytest

K1, K2, K3 = 2.0 ** -17, 2.0 ** -20, 2.0 ** -28      # enc_record's shares
MAX, UNIT, OUT = 8.0, 64.0, -60000.0
G = np.array([-2.0, -2.0, -2.0, 4.0, 4.0, 4.0, -4.0])


def record(M, c, s, inv_l):
    u = np.concatenate([M, c, s[:, None]], axis=1) * inv_l
    m2 = np.sum(u[:, :3] ** 2, axis=1)
    c2 = 2.0 * np.sum(u[:, 3:] ** 2, axis=1)
    nn = m2 + c2
    al = (m2 - c2 - (K1 * nn + K2 * np.sqrt(nn) + K3)) * UNIT
    inside = np.all(np.abs(u) <= MAX, axis=1)
    hi = np.where(inside[:, None], u, 0.0).astype(np.float16)
    lo = (np.where(inside[:, None], u, 0.0) - hi.astype(np.float64)).astype(np.float16)
    al = np.where(inside, al, OUT)
    ahi = al.astype(np.float16)
    alo = np.where(inside, al - ahi.astype(np.float64), 0.0).astype(np.float16)
    return [t.astype(np.float64) for t in (hi, lo, ahi, alo)]


def phi(ri, rj, pessimistic):
    """The filter's value (candidate: below zero), pushed up by the worst summation error."""
    hi, li, ai, bi = ri
    hj, lj, aj, bj = rj
    terms = [G * hi * hj, G * li * hj, G * hi * lj, G * li * lj]
    al_i = np.float32((np.float32(ai) + np.float32(bi)) * np.float32(1.0 / UNIT)).astype(np.float64)
    rest = [aj / UNIT, bj / UNIT, al_i]
    val = sum(np.sum(t, axis=1) for t in terms) + sum(rest)
    mag = sum(np.sum(np.abs(t), axis=1) for t in terms) + sum(np.abs(t) for t in rest)
    return val + (2.0 ** -21 * mag if pessimistic else 0.0)


def pairs(rng, n, lo, hi, scale_c, scale_b):
    """Bodies i anywhere in the shell [lo, hi], bodies j at `t` times the boundary distance."""
    d = rng.normal(size=(n, 3)); d /= np.linalg.norm(d, axis=1)[:, None]
    Mi = d * (10.0 ** rng.uniform(np.log10(lo), np.log10(hi), n))[:, None]
    ci = rng.normal(size=(n, 3)) * scale_c
    cj = ci + rng.normal(size=(n, 3)) * scale_c * (10.0 ** rng.uniform(-4, 0, n))[:, None]
    b = 10.0 ** rng.uniform(-7, np.log10(scale_b), (4, n))
    S = b[0] + b[1] + np.maximum(b[2], b[3])
    bound = np.sqrt(2.0 * np.sum((cj - ci) ** 2, axis=1) + 2.0 * S * S)
    e = rng.normal(size=(n, 3)); e /= np.linalg.norm(e, axis=1)[:, None]
    t = np.where(rng.random(n) < 0.5, 1.0, rng.uniform(0.99, 1.0, n))
    Mj = Mi + e * (bound * t)[:, None]
    return (Mi, ci, b[0] + b[2]), (Mj, cj, b[1] + b[3])


@pytest.mark.parametrize("lo,hi,scale_c,scale_b", [(1.0, 3.0, 0.3, 0.02), (0.5, 5.0, 0.01, 0.005),
                                                   (0.9, 1.1, 0.25, 0.05), (1e-3, 7.9, 0.5, 1e-3),
                                                   (0.01, 0.02, 1e-3, 1e-5)])
def test_no_flaggable_pair_is_dropped(lo, hi, scale_c, scale_b):
    rng = np.random.default_rng(11)
    i, j = pairs(rng, 40000, lo, hi, scale_c, scale_b)
    for unit in (1.0, 0.5, 2.0 ** -3):          # 1/L: the system's largest distance and larger units
        p = phi(record(*i, unit), record(*j, unit), True)
        assert np.all(p < 0.0), (unit, p.max())


def test_body_outside_the_unit_is_always_a_candidate():
    rng = np.random.default_rng(12)
    i, j = pairs(rng, 2000, 1.0, 8.0, 0.3, 0.02)
    far = (i[0] * 100.0, i[1], i[2])
    assert np.all(phi(record(*far, 1.0), record(*j, 1.0), True) < 0.0)
    assert np.all(phi(record(*far, 1.0), record(*far, 1.0), True) < 0.0)


def test_distant_pairs_are_dropped():
    rng = np.random.default_rng(13)
    i, j = pairs(rng, 20000, 1.0, 3.0, 0.05, 0.005)
    # 0.3 length units beyond the boundary
    e = j[0] - i[0]
    e /= np.linalg.norm(e, axis=1)[:, None]
    out = (j[0] + 0.3 * e, j[1], j[2])
    assert np.all(phi(record(*i, 0.25), record(*out, 0.25), False) > 0.0)
