"""What a context's workspace holds: as many sets of drift outputs as fit the bytes set
aside for them, and the persistent launch's records only where it is asked for."""
import ctypes

import numpy as np
import pytest

from paper_2601_19654_amd import nb


def _size(n, nbig=None, **kw):
    p = nb.default_params(**kw)
    off = np.array([0, n], np.int32)
    big = None if nbig is None else np.array([nbig], np.int32)
    out = ctypes.c_size_t()
    assert nb.lib().nb_workspace_size(ctypes.byref(p), 1, off.ctypes.data_as(ctypes.c_void_p),
                                      None if big is None else big.ctypes.data_as(ctypes.c_void_p), 1,
                                      ctypes.byref(out)) == 0
    return out.value


@pytest.mark.parametrize("n,nbig,rec,sets", [
    (1200000, 5000, 0, 8),       # sorted check: 13 doubles a body and set, 7 more sets in 0.81 GiB
    (1500000, 5000, 0, 2),       # 1.02 GiB: two sets
    (980000, 100, 48, 8),        # direct check: its record too, 0.97 GiB
    (1020000, 100, 48, 2)])
def test_sets_of_drift_outputs(n, nbig, rec, sets):
    """Against the full method's context, which holds two sets (and its few rows here)."""
    more = _size(n, nbig) - _size(n, nbig, resolve=1)
    assert abs(more - (sets - 2) * n * (104 + rec)) < 1 << 20


def test_persistent_records_only_where_asked_for():
    n = 8000
    assert abs(_size(n, step_algo=2) + 6 * n * 152 - _size(n, step_algo=1) - 32 * n) < 1 << 16
