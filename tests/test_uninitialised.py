"""No field of the runtime's parameters is left to chance: the host runtime, built once
more with every automatic variable that nothing initialises filled with a pattern, asks
for the workspaces the library asks for."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2601_19654_amd import build, nb


@pytest.fixture(scope="module")
def patterned(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("pattern") / "libruntime.so")
    subprocess.check_call(
        [build.hipcc(), "--offload-arch=" + build.ARCH, "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
         "-ftrivial-auto-var-init=pattern", "-fno-elide-constructors", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-o", out,
         os.path.join(build.CSRC, "nb_runtime.hip"), os.path.join(build.CSRC, "nb_resolve.cpp")])
    nb.lib()                            # (the HIP runtime, loaded the library's way)
    return ctypes.CDLL(out, mode=os.RTLD_LAZY)      # the launchers stay unresolved


def _size(L, n, nsys, nbig, **kw):
    p = nb.default_params(**kw)
    off = (np.arange(nsys + 1) * n).astype(np.int32)
    big = None if nbig is None else np.full(nsys, nbig, np.int32)
    out = ctypes.c_size_t()
    L.nb_workspace_size.restype = ctypes.c_int
    code = L.nb_workspace_size(ctypes.byref(p), nsys, off.ctypes.data_as(ctypes.c_void_p),
                               None if big is None else big.ctypes.data_as(ctypes.c_void_p), 1 << 14, ctypes.byref(out))
    assert code == 0
    return out.value


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n,nsys,nbig,kw", [
    (100, 1, None, {}), (5000, 3, None, {}), (20000, 1, None, {}), (60000, 1, None, {}), (20000, 1, None, {"resolve": 1}),
    (20000, 1, None, {"enc_algo": 1}), (20000, 1, None, {"enc_algo": 4}), (50000, 1, 100, {}), (20000, 1, 15000, {})])
def test_workspace_of_a_patterned_build(patterned, mode, n, nsys, nbig, kw):
    assert _size(patterned, n, nsys, nbig, mode=mode, **kw) == _size(nb.lib(), n, nsys, nbig, mode=mode, **kw)


@pytest.mark.parametrize("n,algo", [(5000, 1), (60000, 2)])
def test_automatic_check_is_the_one_of_the_size(patterned, n, algo):
    for L in (patterned, nb.lib()):
        assert _size(L, n, 1, None, mode=0) == _size(L, n, 1, None, mode=0, enc_algo=algo)
