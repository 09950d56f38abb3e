"""The symmetric FP32C force on both sides of the line between two waves and one per pair
of 128-body tiles (103 tiles, 5356 pairs; 104 tiles, 5460), against the oracle at the
force's bar (1e-6 A_i, A_i the sum of the pair terms' magnitudes)."""
import pytest

import workloads
from gpu_common import accel_error, ctx_for, oracle_dh, pair_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo", [2, 4])
@pytest.mark.parametrize("n", [13184, 13185])
def test_force(n, algo):
    w = workloads.ring(n, m=1e-9)
    _, _, _, a = oracle_dh(w)
    Q = w.x
    c = ctx_for(w, mode=1, force_r=2, force_algo=algo, force_g=1)
    err = accel_error(c.accel(), a, pair_scale(w.m, Q, w.G))
    c.close()
    assert err <= 1e-6, err
