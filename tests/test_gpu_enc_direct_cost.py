"""What the direct encounter check may cost where its filter could stop filtering, with
the lists unchanged."""
import numpy as np
import pytest

import workloads
from gpu_common import ctx_for

pytestmark = pytest.mark.gpu


def _check(w, algo, dt, **kw):
    """Milliseconds of one check after a drift (the least of several), and its list."""
    from paper_2601_19654_amd import nb
    c = ctx_for(w, enc_algo=algo, enc_cap=1 << 20, **kw)
    c.drift(dt)
    e = c.encounters()
    ms = min(c.time_kernel(nb.NB_K_ENCOUNTER, 10) for _ in range(5))
    c.close()
    return ms, e


def _same(a, b):
    return a.nce == b.nce and np.array_equal(a.ice, b.ice) and np.array_equal(a.jce, b.jce) and \
        np.array_equal(a.ce, b.ce)


@pytest.mark.parametrize("far", [1e3, 6.5e4, 1e8])
def test_one_body_far_out(far):
    """One body far from the others: the check of the others costs what it did (46 times
    as much with a unit of length that grows with the largest distance)."""
    w = workloads.ring(9990, m=1e-9)
    base, _ = _check(w, 1, w.dt)
    w.x[4321] *= far
    w.v[4321] /= np.sqrt(far)
    ms, e = _check(w, 1, w.dt)
    _, ref = _check(w, 2, w.dt)
    assert e.nce > 0 and _same(e, ref)
    assert ms < 2.0 * base, (ms, base)


@pytest.mark.parametrize("n,dt", [(500, 0.16), (1001, 0.3), (9990, 0.1), (9990, 0.16)])
def test_long_steps(n, dt):
    """Steps of most of a radian, where the filter keeps most pairs of a ring: the direct
    check costs no more than the sorted one (up to three times as much when every kept
    pair takes the exact test from memory)."""
    w = workloads.ring(n, m=1e-9)
    ms, e = _check(w, 1, dt)
    ref_ms, ref = _check(w, 2, dt)
    print(n, dt, ms, ref_ms)
    assert _same(e, ref)
    assert ms < 1.1 * ref_ms, (ms, ref_ms)
