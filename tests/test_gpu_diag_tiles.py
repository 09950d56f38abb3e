"""Diagnostics at the edges of their tiles (256 targets by 256 sources, sources in
groups of four) against the oracle; tolerance as everywhere for E, E_K, L: 1e-13
relative (FP64 sums with error-free accumulation; each pair term is good to a
few ulp)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_common import ctx_for, oracle_dh, systems

pytestmark = pytest.mark.gpu


def _check(w):
    Q, V, rc, _ = oracle_dh(w)
    c = ctx_for(w)
    # plane-major (3, n): a (3, 3) array is taken as that
    c.upload(w.m0, w.m, np.ascontiguousarray(w.x.T), np.ascontiguousarray(w.v.T))
    d = c.diagnostics()
    for s, lo, hi in systems(w):
        if hi == lo:
            continue
        ref = oracle.energy(w.G, w.m0[s], w.m[lo:hi], Q[lo:hi], V[lo:hi], rc[lo:hi])
        for k in ("E", "EK"):
            assert abs(d[k][s] - ref[k]) <= 1e-13 * abs(ref[k]), (s, k)
        assert np.max(np.abs(d["L"][s] - ref["L"])) <= 1e-13 * np.linalg.norm(ref["L"])
    c.close()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 255, 256, 257, 511, 513, 770])
def test_tile_edges(n):
    # heavy bodies in a narrow ring: pairs inside the changeover zone in every tile
    _check(workloads.ring(n, m=3e-8))


def test_coincident_and_many_systems():
    w = workloads.batch([300, 1, 0, 259, 64, 513])
    w.x[7] = w.x[200]          # the same tile
    w.x[12] = w.x[290]         # another tile
    _check(w)
