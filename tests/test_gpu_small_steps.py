"""Persistent steps of small systems (the automatic step launch up to 256 bodies)
against the oracle and against the per-phase launches, at the edges of waves and
slices.  Tolerances: those of the per-phase steps over a few steps (FP64 1e-11 of
the oracle; FP32C 1e-7, its force at the upload being the FP32C kernel's);
encounter lists and statistics equal."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_common import ctx_for, rel_rows

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2601_19654_amd.nb")

SIZES = [1, 2, 4, 5, 31, 63, 64, 65, 100, 127, 128, 129, 171, 255, 256]


def _up(w, **kw):
    c = ctx_for(w, **kw)
    # plane-major: (3, 3) would be ambiguous
    c.upload(w.m0, w.m, np.ascontiguousarray(w.x.T), np.ascontiguousarray(w.v.T))
    return c


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_matches_oracle_and_launches(n, mode):
    w = workloads.ring(n, m=1e-7)
    c, p = _up(w, mode=mode), _up(w, mode=mode, step_algo=1)
    assert c.choices()["step_algo"] == 2 and p.choices()["step_algo"] == 1
    st = oracle.State.from_workload(w)
    k = 6
    s, sp = c.step(w.dt, k), p.step(w.dt, k)
    total = 0
    for _ in range(k):
        st.step(w.dt)
        total += sum(e[0] for e in st.enc)
    x, v = c.download(nb.NB_DH)
    tol = 1e-11 if mode == 0 else 1e-7
    assert rel_rows(x, st.Q) <= tol and rel_rows(v, st.V) <= 10 * tol
    assert s["total_nce"] == total
    if c.choices()["force_algo"] != p.choices()["force_algo"]:
        # (the tuning table's ordered force counts each pair twice and the bodies themselves)
        s.pop("near_pairs"), sp.pop("near_pairs")
    if mode == 0:
        assert s == sp
    e, ep = c.last_encounters(), p.last_encounters()
    assert np.array_equal(e.ice, ep.ice) and np.array_equal(e.jce, ep.jce) and np.array_equal(e.ce, ep.ce)
    # the drift outputs of the last step are kept: the check on them gives its list
    c.time_kernel(nb.NB_K_ENCOUNTER, reps=1)
    e2 = c.last_encounters()
    assert np.array_equal(e.ice, e2.ice) and np.array_equal(e.jce, e2.jce)


@pytest.mark.parametrize("w", [workloads.batch([1, 0, 17, 128, 64, 65, 2]), workloads.batch([256, 3, 200, 129]),
                               workloads.bigsmall(5, 120, nsys=3, m_big=1e-5, a_lo=0.9, a_hi=1.1), workloads.c2(99)],
                         ids=["batch128", "batch256", "bigsmall", "drag"])
def test_systems_small_bodies_and_drag(w):
    c = ctx_for(w)
    assert c.choices()["step_algo"] == 2
    st = oracle.State.from_workload(w)
    c.step(w.dt, 4)
    for _ in range(4):
        st.step(w.dt)
    x, v = c.download(nb.NB_DH)
    assert rel_rows(x, st.Q) <= 1e-11 and rel_rows(v, st.V) <= 1e-10


@pytest.mark.parametrize("w", [workloads.ring(150, m=1e-7), workloads.c2(80)], ids=["ring", "drag"])
def test_runs_of_any_length_give_the_same_bits(w):
    a, b = ctx_for(w), ctx_for(w)
    a.step(w.dt, 300)
    for k in (1, 7, 256, 36):
        b.step(w.dt, k)
    for p, q in zip(a.download(nb.NB_DH), b.download(nb.NB_DH)):
        assert np.array_equal(p, q)
    assert np.array_equal(a.accel(), b.accel()) and np.array_equal(a.rcrit(), b.rcrit())


def test_events_after_small_steps():
    w = workloads.ring(200, m=1e-6)
    out = []
    for sa in (0, 1):
        c = ctx_for(w, step_algo=sa)
        c.step(w.dt, 3)
        out.append(c.events(1e4, 0.0, 1.05)[0])
        idx = c.compact()
        c.step(w.dt, 2)
        out[-1]["kept"] = len(idx)
        c.close()
    assert out[0] == out[1] and out[0]["ejected"] > 0
