"""How the binding hands arrays to the library (CPU only): writable, read-only, strided and empty ones arrive alike."""
import ctypes as C

import numpy as np
import pytest

from paper_1906_00148_amd import binding as B


@pytest.mark.parametrize("dtype,ty", [(np.uint8, C.c_uint8), (np.int8, C.c_int8), (np.uint32, C.c_uint32), (np.int32, C.c_int32)])
def test_an_array_is_passed_by_its_address(dtype, ty):
    L = C.CDLL(None)
    L.memcmp.restype, L.memcmp.argtypes = C.c_int, [C.POINTER(ty), C.c_void_p, C.c_size_t]
    a = np.arange(24, dtype=dtype).reshape(4, 6)
    read_only = a.copy()
    read_only.flags.writeable = False
    for v in (a, a[1:], a[2:3, 1:4], a[:, 1:4], a[::2], read_only, read_only[0], np.frombuffer(a.tobytes(), dtype)):
        assert L.memcmp(B._p(v, ty), v.ctypes.data, v.itemsize * v.shape[-1]) == 0
    scratch = np.zeros(4, dtype)
    L.memset.argtypes = [C.POINTER(ty), C.c_int, C.c_size_t]
    L.memset(B._p(scratch, ty), 1, scratch.nbytes)
    assert np.all(scratch.view(np.uint8) == 1)
    B._p(np.zeros(0, dtype), ty)


def test_plans_of_read_only_weights():
    sign, exp = np.array([[1, -1, 1]], np.int8), np.array([[0, -2, -7]], np.int8)
    want = B.plan_shift_acc(1, 3, 8, sign, exp, 12)
    sign.flags.writeable = exp.flags.writeable = False
    assert B.plan_shift_acc(1, 3, 8, sign, exp, 12) == want
