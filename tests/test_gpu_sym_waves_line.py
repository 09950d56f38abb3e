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


@pytest.mark.parametrize("g", [2, 4])
@pytest.mark.parametrize("n", [700, 1031])
def test_radial_order_in_wider_workgroups(n, g):
    """Over the radial order wider workgroups keep the sources' run sums in LDS."""
    w = workloads.ring(n, m=1e-7)
    _, _, _, a = oracle_dh(w)
    c = ctx_for(w, mode=1, force_r=2, force_algo=4, force_g=g)
    err = accel_error(c.accel(), a, pair_scale(w.m, w.x, w.G))
    c.close()
    assert err <= 1e-6, err


@pytest.mark.parametrize("mode,algo,n", [(1, 2, 13800), (1, 4, 16500), (0, 2, 22500)])
def test_check_in_workgroups_of_several_waves(mode, algo, n):
    """Beside one wave per tile pair the sorted check's pair test runs in workgroups of two
    or four waves: after steps in a run, the list of the direct check from the same arcs."""
    lists = []
    for enc in (1, 2):
        w = workloads.ring(n, m=1e-9)
        c = ctx_for(w, mode=mode, force_r=2, force_algo=algo, force_g=1, enc_algo=enc)
        st = c.step(w.dt, 3)
        e = c.last_encounters()
        lists.append((st["total_nce"], e.nce, e.ice.tolist(), e.jce.tolist(), e.ce.tolist()))
        c.close()
    assert lists[0] == lists[1] and lists[0][1] > 0
