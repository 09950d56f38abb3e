"""Contexts that lose bodies: all of them, and as many as take the automatic choices
past their lines."""
import numpy as np
import pytest

import workloads
from gpu_common import ctx_for

pytestmark = pytest.mark.gpu


def _lose(c, w, lost):
    """Eject the first `lost` bodies of w (unbound and beyond the ejection radius)."""
    c.step(w.dt, 1)
    cnt, _ = c.events(1e12, 0.0, 50.0)
    assert cnt["ejected"] == lost
    return c.compact()


def _far(w, lost):
    w.x[:lost] *= 100.0
    w.v[:lost] *= 3.0
    return w


@pytest.mark.parametrize("step_algo", [0, 1])
@pytest.mark.parametrize("n,kw", [(40, {}), (300, {}), (300, {"mode": 1}), (300, {"resolve": 1}),
                                  (300, {"enc_algo": 2})])
def test_context_without_bodies(n, kw, step_algo):
    """Every body lost: steps, phases, lists and diagnostics still run, on nothing."""
    from paper_2601_19654_amd import nb
    w = _far(workloads.ring(n), n)
    c = ctx_for(w, step_algo=step_algo, **kw)
    idx = _lose(c, w, n)
    assert len(idx) == 0 and c.ntot == 0
    for steps in (1, 11):
        st = c.step(w.dt, steps)
        assert st["total_nce"] == 0 and st["kepler_fail"] == 0
    assert c.last_encounters().nce == 0
    c.drift(w.dt)
    assert c.encounters().nce == 0
    c.force()
    c.kick(w.dt)
    assert np.all(c.diagnostics()["E"] == 0.0)
    x, _ = c.download(nb.NB_DH)
    assert x.shape[0] == 0
    c.close()
