"""The workspace the reverse step keeps: what its kernels fill and nothing more.

1-D: two face states of six numbers and their adjoints for each of the nx + 2 extended
cells, one sum for each of the nx + 4 padded positions; 2-D: none.  That these suffice
is checked by the reverse pass on the CPU in a buffer of this size (test_adjoint_host,
with the sanitizers too).
"""
import re
import subprocess

import ctypes

import paper_1210_5246_amd as csh


def test_workspace_size():
    names = subprocess.run(["nm", "-D", csh.LIB_PATH], capture_output=True, text=True, check=True).stdout
    name = re.search(r"\b(_Z\w*csh_adjoint_workspace_doubles\w*)", names).group(1)
    f = getattr(csh.lib(), name)
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int, ctypes.c_int]
    for nx in (1, 2, 61, 4096, 1 << 28):
        assert f(nx, 1) == 2 * 2 * 6 * (nx + 2) + 6 * (nx + 4)
        assert f(nx, 2) == 0
