"""The direct encounter check's list against the oracle's: at the edges of its strips
of 128 targets, groups of 16 rows and source chunks, with short steps (few candidates)
and with steps of most of a radian (most pairs candidates), over one set of drift arcs
(the oracle's drift differs from the device's by rounding: pairs within 1e-9 of the
threshold may fall either way)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_common import ctx_for, nbig_of, oracle_dh, systems

pytestmark = pytest.mark.gpu


def _expected(w, dt):
    """(sure, allowed): pairs that must be listed, and those that may be."""
    Q0, V0, rc, _ = oracle_dh(w)
    sure, allowed = set(), set()
    for s, lo, hi in systems(w):
        if hi == lo:
            continue
        q0, v0 = Q0[lo:hi], V0[lo:hi]
        q1, v1, _ = oracle.drift(w.G * w.m0[s], dt, q0, v0)
        nb_ = nbig_of(w, s)
        for out, f in ((sure, 1 - 1e-9), (allowed, 1 + 1e-9)):
            e = oracle.encounters(dt, q0, v0, q1, v1, rc[lo:hi] * f, nbig=nb_)
            out.update(zip((e["ice"] + lo).tolist(), (e["jce"] + lo).tolist()))
    return sure, allowed


def _check(w, dt, **kw):
    sure, allowed = _expected(w, dt)
    c = ctx_for(w, enc_cap=1 << 18, **kw)
    c.drift(dt)
    e = c.encounters()
    got = set(zip(e.ice.tolist(), e.jce.tolist()))
    assert len(got) == e.nce and sure <= got <= allowed
    ends = {i for p in got for i in p}
    assert ends == set(np.nonzero(e.ce)[0].tolist())
    c.close()
    return len(got)


@pytest.mark.parametrize("dt", [0.04, 0.2, 0.6])
@pytest.mark.parametrize("n", [2, 16, 17, 63, 64, 65, 127, 128, 129, 193, 300, 513])
def test_edges(n, dt):
    count = _check(workloads.ring(n, m=1e-6), dt, enc_algo=1)
    assert count > 0 or n < 65      # (the oracle lists none of some smaller rings)


@pytest.mark.parametrize("jchunk", [0, 16, 48, 128, 1024])
@pytest.mark.parametrize("dt", [0.04, 0.3])
def test_chunks(jchunk, dt):
    assert _check(workloads.ring(301, m=1e-6), dt, enc_algo=1, enc_jchunk=jchunk) > 0


@pytest.mark.parametrize("nb_,ns", [(1, 300), (17, 300), (100, 333), (130, 200)])
@pytest.mark.parametrize("dt", [0.04, 0.3])
def test_big_and_small(nb_, ns, dt):
    w = workloads.bigsmall(nb_, ns, nsys=2, a_lo=0.95, a_hi=1.05, m_big=1e-5)
    assert _check(w, dt, enc_algo=3 if nb_ <= 256 else 1) > 0


@pytest.mark.parametrize("dt", [0.04, 0.3])
def test_systems(dt):
    w = workloads.batch([3, 260, 0, 64, 65, 1, 129, 300])
    w.m[:] = 3e-7
    assert _check(w, dt, enc_algo=1) > 0
