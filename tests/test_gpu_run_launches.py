"""Steps inside a captured run leave launches out (the force's partials are summed
by the next step's drift launch, with gas drag by the kick, whose sums of m V the steps
hand on; the direct checks of a run are counted at its end): the same bits and the same lists and statistics as single steps, which are
runs of one step, at the slot counts where the summing changes (8, 16, 32, 64
slots), for batches, small bodies and both modes."""
import dataclasses

import numpy as np
import pytest

import workloads
from gpu_common import ctx_for

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2601_19654_amd.nb")


def _check(w, **kw):
    a, b = ctx_for(w, **kw), ctx_for(w, **kw)
    for k in (8, 11, 3):
        sa = a.step(w.dt, k)
        sb = [b.step(w.dt, 1) for _ in range(k)]
        for key in ("total_nce", "near_pairs", "kepler_fail", "overflow_steps"):
            assert sa[key] == sum(s[key] for s in sb), key
        assert sa["max_nce"] == max(s["max_nce"] for s in sb)
        ea, eb = a.last_encounters(), b.last_encounters()
        assert np.array_equal(ea.ice, eb.ice) and np.array_equal(ea.jce, eb.jce)
        assert np.array_equal(ea.ce, eb.ce)
    for p, q in zip(a.download(nb.NB_DH), b.download(nb.NB_DH)):
        assert np.array_equal(p, q)
    assert np.array_equal(a.accel(), b.accel())
    return sa["total_nce"]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n", [300, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_slot_counts(n, mode):
    # tiles of 64 bodies: 5 .. 65 slots
    assert _check(workloads.ring(n, m=3e-7), mode=mode, step_algo=1, force_r=1, force_g=1) > 0


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n", [300, 512, 513, 1025, 4096, 4097])
def test_drag(n, mode):
    w = dataclasses.replace(workloads.ring(n, m=3e-7), drag=True)
    kw = dict(mode=mode, step_algo=1, force_r=1, force_g=1, force_algo=2)
    _check(w, **kw)
    # against the phases, which sum the partials and m V in launches of their own
    a, b = ctx_for(w, **kw), ctx_for(w, **kw)
    a.step(w.dt, 3)
    h = 0.5 * w.dt
    for _ in range(3):
        b.kick(h)
        b.sun_drift(h)
        b.drift(w.dt)
        b.encounters()
        b.sun_drift(h)
        b.force()
        b.kick(h)
    for p, q in zip(a.download(nb.NB_DH), b.download(nb.NB_DH)):
        assert np.max(np.abs(p - q)) <= 1e-14 * np.max(np.abs(p))


def test_many_systems():
    # more workgroups than the launches sum partials in with several threads a body
    _check(workloads.batch([560] * 300), mode=1, step_algo=1, force_algo=2)


@pytest.mark.parametrize("w", [workloads.batch([900, 1, 0, 300, 2100]), workloads.bigsmall(40, 3000, m_big=1e-5, a_lo=0.95, a_hi=1.05)],
                         ids=["batch", "bigsmall"])
def test_systems(w):
    _check(w, step_algo=1)


def test_workspace_holding_anything():
    """The flags do not depend on what the workspace held (here the tags a run writes)."""
    import torch
    w = workloads.ring(1500, m=1e-7)
    ref = ctx_for(w, step_algo=1)
    ref.step(w.dt, 8)
    want = ref.last_encounters()
    ref.close()
    real = torch.empty
    try:
        torch.empty = lambda *a, **k: real(*a, **k).view(torch.int32).fill_(23).view(torch.uint8) \
            if k.get("dtype") == torch.uint8 else real(*a, **k)
        c = ctx_for(w, step_algo=1)
    finally:
        torch.empty = real
    c.step(w.dt, 8)
    got = c.last_encounters()
    assert np.array_equal(got.ce, want.ce) and np.array_equal(got.ice, want.ice) and want.nce > 0


def test_uploads_between_runs():
    """Captured runs are kept over an upload: replays after other states and
    other eager work equal a fresh context's."""
    ws = [workloads.ring(700, seed_sys=k, m=1e-7) for k in range(3)]
    c = ctx_for(ws[0])
    for w in ws + ws:
        c.upload(w.m0, w.m, w.x, w.v)
        c.diagnostics()
        c.step(w.dt, 19)
        f = ctx_for(w)
        f.step(w.dt, 19)
        for p, q in zip(c.download(nb.NB_DH), f.download(nb.NB_DH)):
            assert np.array_equal(p, q)
        f.close()
