"""Compactions that take a context past the lines of the automatic choices (targets per
lane, super-tile width, step launch, encounter check, sets of drift outputs): the smaller
layout fits the workspace the context was created with, steps like a fresh context of
the same bodies, and, where the workspace has the room, with the same choices (without
the tuning table, whose rows are those of the size at creation)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _compacted(w, lost, **kw):
    """A context of w after the bodies in `lost` were ejected and removed."""
    w.x[lost] *= 100.0
    w.v[lost] *= 3.0           # unbound, beyond the ejection radius
    from paper_2601_19654_amd import nb
    c = nb.Context(w.off, nb.default_params(G=w.G, **kw), enc_cap=1 << 16, device="cuda:0", tuned=False)
    c.upload(w.m0, w.m, w.x, w.v)
    c.step(w.dt, 1)
    cnt, _ = c.events(1e12, 0.0, 50.0)
    assert cnt["ejected"] == len(lost)
    idx = c.compact()
    assert len(idx) == w.ntot - len(lost) == c.ntot
    return c, idx


def _fresh(w, c, idx, **kw):
    from paper_2601_19654_amd import nb
    x, v = c.download(nb.NB_DH)
    f = nb.Context(c.off, nb.default_params(G=w.G, **kw), enc_cap=1 << 16, device="cuda:0", tuned=False)
    f.upload(w.m0, w.m[idx], x, v, frame=nb.NB_DH)
    return f


def _step_alike(w, c, f, tol):
    from paper_2601_19654_amd import nb
    for t in (c, f):
        t.step(w.dt, 2)
    e, g = c.last_encounters(), f.last_encounters()
    assert e.nce == g.nce and np.array_equal(e.ice, g.ice) and np.array_equal(e.jce, g.jce)
    (x, v), (y, u) = c.download(nb.NB_DH), f.download(nb.NB_DH)
    assert np.max(np.abs(x - y)) <= tol * np.max(np.abs(y))
    assert np.max(np.abs(v - u)) <= tol * np.max(np.abs(u))


@pytest.mark.parametrize("mode,tol", [(0, 1e-11), (1, 1e-7)])
@pytest.mark.parametrize("n,lost,nsys,kw", [
    (33000, 660, 1, {}),                 # super-tiles of 2 -> 1 tiles: twice the partials a body
    (33000, 660, 1, {"resolve": 1}),
    (12000, 1200, 8, {}),                # in every one of several systems
    (4500, 200, 1, {}),                  # two targets per lane -> one
])
def test_smaller_layout_fits(n, lost, nsys, kw, mode, tol):
    w = workloads.batch([n] * nsys)
    w.m[:] = 1e-10
    gone = np.concatenate([np.arange(lost) + s * n for s in range(nsys)])
    c, idx = _compacted(w, gone, mode=mode, **kw)
    f = _fresh(w, c, idx, mode=mode, **kw)
    _step_alike(w, c, f, tol)
    c.close()
    f.close()


@pytest.mark.parametrize("n,lost", [(300, 180), (260, 10), (700, 600)])
def test_small_systems_take_the_small_launch(n, lost):
    """A context that began above the size of the one-workgroup launch steps with it once
    few bodies are left, as a fresh context does."""
    w = workloads.ring(n, m=1e-7)
    c, idx = _compacted(w, np.arange(lost))
    f = _fresh(w, c, idx)
    assert c.choices() == f.choices() and c.choices()["step_algo"] == 2
    _step_alike(w, c, f, 0.0)
    c.close()
    f.close()
