"""Contexts whose matrix elements or primitive pairs of a class do not fit the
32-bit numbers the device tables use are refused before the GPU is touched."""

import ctypes
import os

import numpy as np
import pytest

LIBPATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                       "paper_2510_24968_amd", "libfsim.so")


def _s_shells(n, nprim):
    """n s shells of nprim primitives, all on one atom and of one exponent set."""
    return dict(xyz=np.zeros((1, 3)), Z=np.ones(1), shell_atom=np.zeros(n, np.int32),
                shell_l=np.zeros(n, np.int32), shell_nprim=np.full(n, nprim, np.int32),
                shell_prim0=np.zeros(n, np.int32), exps=np.linspace(0.5, 2.0, nprim),
                coefs=np.ones(nprim), nelec=2)


@pytest.mark.parametrize("nmol,n,nprim,needle", [
    (1, 46341, 1, "packed matrix size 2147488281"),    # 46340^2 < 2^31 < 46341^2
    (2, 32769, 1, "packed matrix size 2147614722"),
    (1, 8192, 8, "33558528 pairs of 64 primitive pairs"),
])
def test_sizes_beyond_32_bits_are_refused(nmol, n, nprim, needle):
    from paper_2510_24968_amd.fsim import _Basis, _Options, basis_struct
    so = ctypes.CDLL(LIBPATH)
    so.fsim_batch_create.restype = so.fsim_ctx_create.restype = ctypes.c_int
    so.fsim_last_error.restype = ctypes.c_char_p
    made = [basis_struct(_s_shells(n, nprim)) for _ in range(nmol)]
    arr = (_Basis * nmol)(*[m[0] for m in made])
    o, h = _Options(0.0, 0.0, 8, 1e-8, 1e-10, 50, 0), ctypes.c_void_p()
    if nmol == 1:
        st = so.fsim_ctx_create(ctypes.byref(arr[0]), ctypes.byref(o), ctypes.byref(h))
    else:
        st = so.fsim_batch_create(arr, nmol, ctypes.byref(o), ctypes.byref(h))
    assert st == -1 and needle in so.fsim_last_error().decode() and not h.value
