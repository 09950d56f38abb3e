"""The direct encounter check (matrix-core filter, then the exact test) against the
sorted check, which shares only the exact test with it: the lists must be equal,
at the edges of its strips of 128 targets, groups of 16 rows and source chunks,
with a body far outside the others, and where a context whose steps run the
sorted check takes the direct one for nb_drift and nb_encounters."""
import numpy as np
import pytest

import workloads
from gpu_common import ctx_for

pytestmark = pytest.mark.gpu


def _list(w, algo, via_step=False, **kw):
    c = ctx_for(w, enc_algo=algo, enc_cap=1 << 18, **kw)
    if via_step:
        c.step(w.dt, 2)
        e = c.last_encounters()
    else:
        c.drift(w.dt)
        e = c.encounters()
    choice = c.choices()["enc_algo"]
    c.close()
    return e, choice


def _same(w, a, b, **kw):
    (ea, _), (eb, _) = _list(w, a, **kw), _list(w, b, **kw)
    assert ea.nce == eb.nce
    assert np.array_equal(ea.ice, eb.ice) and np.array_equal(ea.jce, eb.jce)
    assert np.array_equal(ea.ce, eb.ce)
    return ea.nce


@pytest.mark.parametrize("n", [2, 15, 16, 17, 127, 128, 129, 145, 257, 513, 1031, 2048])
def test_edges(n):
    # heavy bodies: many encounters also in a small ring
    _same(workloads.ring(n, m=1e-6), 1, 2)


@pytest.mark.parametrize("jchunk", [16, 128, 100, 4096])
def test_chunks_and_systems(jchunk):
    w = workloads.batch([3, 700, 0, 64, 65, 1, 129, 300])
    w.m[:] = 3e-7
    assert _same(w, 1, 2, enc_jchunk=jchunk) > 0


@pytest.mark.parametrize("nb_,ns", [(1, 600), (17, 1000), (100, 5000), (130, 777)])
def test_big_and_small(nb_, ns):
    w = workloads.bigsmall(nb_, ns, nsys=2, a_lo=0.95, a_hi=1.05, m_big=1e-5)
    assert _same(w, 3 if nb_ <= 256 else 1, 2) > 0


def test_body_far_outside():
    w = workloads.ring(1200, m=1e-6)
    w.x[5] *= 40.0
    w.x[77] *= 1e4
    w.v[5] /= np.sqrt(40.0)
    w.v[77] /= 100.0
    assert _same(w, 1, 2) > 0


def test_alone_and_beside_the_step():
    w = workloads.ring(12000, m=1e-9)
    (ea, ca), (eb, cb) = _list(w, 0), _list(w, 2)
    assert ca == cb == 2 and ea.nce == eb.nce > 0
    assert np.array_equal(ea.ice, eb.ice) and np.array_equal(ea.jce, eb.jce) and np.array_equal(ea.ce, eb.ce)
    (ea, _), (eb, _) = _list(w, 0, True), _list(w, 1, True)
    assert ea.nce == eb.nce > 0
    assert np.array_equal(ea.ice, eb.ice) and np.array_equal(ea.jce, eb.jce) and np.array_equal(ea.ce, eb.ce)


@pytest.mark.parametrize("n,lost", [(10030, 60), (10200, 700), (41000, 300)])
def test_compaction_past_the_line(n, lost):
    """A compaction takes a context past the line between the checks: it still fits the
    workspace it was created with, and its next list is a fresh context's."""
    from paper_2601_19654_amd import nb
    w = workloads.ring(n, m=1e-9)
    w.x[:lost] *= 100.0
    w.v[:lost] *= 3.0          # unbound, beyond the ejection radius
    c = ctx_for(w, step_algo=1)
    c.step(w.dt, 1)
    cnt, _ = c.events(1e12, 0.0, 50.0)
    assert cnt["ejected"] == lost
    idx = c.compact()
    assert len(idx) <= n - lost and c.ntot == len(idx)
    x, v = c.download(nb.NB_DH)
    c.step(w.dt, 1)
    e = c.last_encounters()
    f = nb.Context(c.off, nb.default_params(G=w.G, step_algo=1), enc_cap=1 << 16, device="cuda:0")
    f.upload(w.m0, w.m[idx], x, v, frame=nb.NB_DH)
    f.step(w.dt, 1)
    g = f.last_encounters()
    assert e.nce == g.nce and np.array_equal(e.ice, g.ice) and np.array_equal(e.jce, g.jce)
    c.close()
    f.close()
