"""The unit of length of the direct encounter check's records: a typical distance of
the system's bodies, the midpoints outside a ball of 7.5 units moved to its nearest
point.  No pair that can be flagged may be dropped (the records emulated as in
test_enc_matrix_bound, which this file's emulation extends), and one body far out may
not make candidates of the others' pairs."""
import numpy as np
import pytest

from test_enc_matrix_bound import pairs, phi, record

BALL = 7.5


def clamped(M, c, d, s, inv_l):
    r = np.linalg.norm(M, axis=1) * inv_l
    return record(M * np.where(r > BALL, BALL / np.maximum(r, 1e-300), 1.0)[:, None], c, d, s, inv_l)


def inv_unit(Q):
    """1/L from the mean binary exponent of |Q|^2."""
    e = np.floor(np.log2(np.sum(Q ** 2, axis=1))).astype(int)
    return 2.0 ** -((int(np.floor(e.sum() / len(e))) >> 1) + 1)


@pytest.mark.parametrize("lo,hi", [(1.0, 3.0), (1.0, 1e3), (6.0, 9.0), (7.0, 1e6), (1e4, 1e7)])
@pytest.mark.parametrize("scale_c,scale_d,scale_s", [(0.3, 0.02, 0.02), (0.01, 1e-4, 0.005), (1.5, 1.0, 0.5)])
def test_no_flaggable_pair_is_dropped(lo, hi, scale_c, scale_d, scale_s):
    rng = np.random.default_rng(31)
    i, j = pairs(rng, 20000, lo, hi, scale_c, scale_d, scale_s)
    for inv_l in (1.0, 0.25):
        p = phi(clamped(*i, inv_l), clamped(*j, inv_l), True)
        assert np.all(p < 0.0), (inv_l, p.max())


@pytest.mark.parametrize("far", [30.0, 1e3, 1e5, 1e9])
def test_a_far_body_leaves_the_others_pairs_alone(far):
    """The share of candidates of a 1-3 AU disk with short chords does not grow with
    the distance of one body; the far body meets those at the ball's edge alone."""
    rng = np.random.default_rng(32)
    n = 800
    phi_ = rng.uniform(0, 2 * np.pi, n)
    r = rng.uniform(1.0, 3.0, n)
    M = np.stack([r * np.cos(phi_), r * np.sin(phi_), 0.01 * rng.normal(size=n)], axis=1)
    c = 0.3 * np.stack([-np.sin(phi_), np.cos(phi_), np.zeros(n)], axis=1) / np.sqrt(r)[:, None]
    d = -0.04 * M / r[:, None] ** 3
    s = np.full(n, 2e-3)

    def share(M):
        inv_l = inv_unit(M)
        i, j = np.triu_indices(n, 1)
        rec = clamped(M, c, d, s, inv_l)
        cand = phi(tuple(t[i] for t in rec), tuple(t[j] for t in rec), False) < 0.0
        return cand.sum(), (cand & (i == 0)).sum()

    base, _ = share(M)
    M[0] *= far / r[0]
    c[0] = d[0] = 0.0
    most, own = share(M)
    assert own == 0 and most <= base + 8


def test_unit_is_a_typical_distance():
    rng = np.random.default_rng(33)
    Q = rng.normal(size=(4000, 3))
    Q *= (rng.uniform(1.0, 3.0, 4000) / np.linalg.norm(Q, axis=1))[:, None]
    assert inv_unit(Q) == 0.5
    Q[7] *= 1e6
    assert inv_unit(Q) == 0.5
    assert inv_unit(1e-9 * Q) == 0.5 * 2.0 ** 30
