"""The arguments of a state read, checked before the library is entered (no GPU)."""
import ctypes as C

import numpy as np
import pytest

from paper_2609_02675_amd import _lib


@pytest.mark.parametrize("call", ["scene", "batch"])
def test_state_arrays_are_doubles(call):
    """A state read takes pointers to doubles (or untyped ones); an array of another
    type, which the library would write past, is refused before the call."""
    fn = getattr(_lib.lib(), f"pabd_{call}_read_state")
    head = (None,) if call == "scene" else (None, 0)
    doubles, floats = np.zeros(12), np.zeros(12, np.float32)
    for ok in (None, doubles.ctypes.data_as(C.POINTER(C.c_double)), doubles.ctypes.data_as(C.c_void_p), (C.c_double * 12)()):
        assert fn(*head, ok, None, None, None) == _lib.PABD_E_INVALID  # a null handle
    for bad in (floats.ctypes.data_as(C.POINTER(C.c_float)), (C.c_float * 12)(), doubles.ctypes.data, doubles):
        with pytest.raises(C.ArgumentError):
            fn(*head, bad, None, None, None)
