"""The FP32 form of the exact encounter test's Hermite bound, to which the direct check
puts every pair of a group whose matrix filter keeps most of them: it passes every pair
the exact test can flag (emulated in float32, operation by operation, against the
oracle's exact minimum and against the bound in float64)."""
import numpy as np
import pytest

import oracle
import workloads

F = np.float32


def record(dt, q0, v0, q1, v1, rc, inv_l):
    q0, q1, c, d = inv_l * q0, inv_l * q1, inv_l * dt * v0, inv_l * dt * v1
    with np.errstate(over="ignore"):
        w = sum(np.sum(t * t, axis=1) for t in (q0, q1, c, d))
    with np.errstate(over="ignore", invalid="ignore"):
        return (q0.astype(F), q1.astype(F), (2 * c).astype(F), (2 * d).astype(F),
                (inv_l * rc * (1 + 2.0 ** -18)).astype(F), (w * (2.0 ** -18 * (1 + 2.0 ** -20))).astype(F))


def passes(ri, rj):
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(F)  # noqa: E731
    with np.errstate(over="ignore", invalid="ignore"):
        a, b, c, d = (rj[k] - ri[k] for k in range(4))
        zero = np.zeros(len(a), F)
        f0, f1, g0, g1 = zero, zero, zero, zero
        for k in range(3):
            f0, f1 = fma(a[:, k], a[:, k], f0), fma(b[:, k], b[:, k], f1)
            g0, g1 = fma(a[:, k], c[:, k], g0), fma(b[:, k], d[:, k], g1)
        s = np.fmax(zero, -g0) + np.fmax(zero, g1)
        lower = fma(np.full(len(s), F(-4.0 / 27.0)), s, np.fmin(f0, f1))
        rc = np.fmax(ri[4], rj[4])
        return ~(lower > fma(rc, rc, ri[5] + rj[5]))


def bound64(dt, bi, bj):
    """The exact test's bound minus its threshold, float64."""
    d0, d1 = bj[0] - bi[0], bj[2] - bi[2]
    f0, f1 = np.sum(d0 * d0, axis=1), np.sum(d1 * d1, axis=1)
    g0 = 2 * dt * np.sum(d0 * (bj[1] - bi[1]), axis=1)
    g1 = 2 * dt * np.sum(d1 * (bj[3] - bi[3]), axis=1)
    rc2 = np.maximum(bi[4], bj[4]) ** 2
    return np.minimum(f0, f1) - 4 / 27 * (np.maximum(0, -g0) + np.maximum(0, g1)) - \
        (rc2 * (1 + 1e-6) + 1e-15 * (f0 + f1 + np.abs(g0) + np.abs(g1)))


@pytest.mark.parametrize("scale", [1.0, 1e-6, 1e12])
@pytest.mark.parametrize("spread", [1.0, 1e-2, 1e-4])
def test_no_pair_the_bound_passes_is_dropped(scale, spread):
    """Random data with rc set so that the float64 bound is met to within rounding."""
    rng = np.random.default_rng(5)
    n, dt = 200000, 0.3
    body = lambda: [rng.normal(size=(n, 3)) for _ in range(4)]  # noqa: E731
    bi = body()
    bj = [x + spread * y for x, y in zip(bi, body())]
    bi, bj = [scale * t for t in bi], [scale * t for t in bj]
    zero = np.zeros(n)
    need = bound64(dt, bi + [zero], bj + [zero])
    rc = np.sqrt(np.maximum(need, 0.0)) * (1 + 1e-12)
    bi, bj = bi + [rc], bj + [np.where(rng.random(n) < 0.5, rc, 0.0)]
    must = bound64(dt, bi, bj) <= 0.0
    assert must.mean() > 0.9
    for inv_l in (1.0 / scale, 0.13 / scale, 8.0 / scale):
        ok = passes(record(dt, *bi, inv_l), record(dt, *bj, inv_l))
        assert np.all(ok[must])


def test_values_out_of_range_pass():
    rng = np.random.default_rng(6)
    q = rng.normal(size=(8, 3))
    big = [np.array([1e30, np.inf, np.nan, 1e38, 1e300, 1e20, 1e25, 3e38])[:, None] * np.ones(3)] * 4
    ri = record(0.1, q, q, q, q, np.ones(8), 1.0)
    rj = record(0.1, *big, np.ones(8), 1.0)
    assert np.all(passes(ri, rj))


@pytest.mark.parametrize("dt", [0.04, 0.16, 0.5])
def test_flagged_pairs_pass_and_few_others_do(dt):
    w = workloads.ring(400, m=1e-7)
    Q0, V0 = oracle.helio_to_dh(1.0, w.m, w.x, w.v)
    rc = oracle.rcrit(1.0, w.m, Q0)
    Q1, V1, _ = oracle.drift(w.G * 1.0, dt, Q0, V0)
    e = oracle.encounters(dt, Q0, V0, Q1, V1, rc)
    r = record(dt, Q0, V0, Q1, V1, rc, 1.0)
    i, j = np.triu_indices(400, 1)
    ok = passes(tuple(t[i] for t in r), tuple(t[j] for t in r))
    kept = {(a, b) for a, b in zip(i[ok].tolist(), j[ok].tolist())}
    flagged = list(zip(e["ice"].tolist(), e["jce"].tolist()))
    assert len(flagged) > 5 and all(p in kept for p in flagged)
    assert dt > 0.2 or len(kept) < 0.05 * len(i)
