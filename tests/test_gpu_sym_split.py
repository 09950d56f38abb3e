"""Tile pairs of the symmetric force shared by several waves of a workgroup: sizes on
both sides of the lines between four, two and one waves per pair, last tiles that
hold a few bodies or none in a sub-tile, ragged batches, index and radial order,
with changeover pairs, against the oracle at the bars of the force (FP64 1e-12 A_i,
FP32C 1e-6 A_i, A_i the sum of the pair terms' magnitudes)."""
import numpy as np
import pytest

import workloads
from gpu_common import accel_error, ctx_for, oracle_dh, pair_scale, systems

pytestmark = pytest.mark.gpu

# tile pairs of 64: 1 (n 64), 3, 1035 (2880 bodies), 1081, 4095 (5760), 4186
# tile pairs of 128: 1, 3, 4095 (11520 bodies), 4186
SIZES = [(1, n) for n in (2, 64, 65, 129, 700, 2880, 2881, 5760, 5800)] + \
        [(2, n) for n in (5, 64, 65, 128, 129, 193, 1031, 11520, 11530)]
_ref = {}


def _case(name):
    if name not in _ref:
        w = workloads.ring(name, m=1e-7) if isinstance(name, int) else \
            workloads.batch([3, 700, 0, 64, 65, 1, 129, 300, 193], cfg_id=31, a_lo=0.95, a_hi=1.05)
        Q, V, rc, a = oracle_dh(w)
        A = [pair_scale(w.m[lo:hi], Q[lo:hi], w.G) if hi - lo > 1 else None for _, lo, hi in systems(w)]
        _ref[name] = w, a, A
    return _ref[name]


def _check(name, mode, r, algo):
    w, a_ref, A = _case(name)
    c = ctx_for(w, mode=mode, force_r=r, force_algo=algo, force_g=1)
    a, b = c.accel(), None
    c.force()
    b = c.accel()
    c.close()
    assert np.array_equal(a, b)
    for s, lo, hi in systems(w):
        if hi - lo < 2:
            assert np.all(a[lo:hi] == 0.0)
            continue
        err = accel_error(a[lo:hi], a_ref[lo:hi], A[s])
        assert err <= (1e-12 if mode == 0 else 1e-6), (name, s, err)


@pytest.mark.parametrize("r,n", SIZES)
@pytest.mark.parametrize("mode,algo", [(0, 2), (1, 2), (1, 4)])
def test_sizes(mode, algo, r, n):
    _check(n, mode, r, algo)


@pytest.mark.parametrize("r", [1, 2])
@pytest.mark.parametrize("mode,algo", [(0, 2), (1, 2), (1, 4)])
def test_ragged(mode, algo, r):
    _check("batch", mode, r, algo)
