"""Arguments of the Python entry points (no GPU needed: every call here ends in a check on the host).  They take what ctypes takes
for the C entry points' argument types, and refuse what it refuses."""
import ctypes as C

import numpy as np
import pytest

import paper_2310_06993_amd.binding as b

BAD_ALIGN = 5


@pytest.fixture
def arr():
    """One bucket whose first pointer is not aligned: whoever reads the right memory answers OR_ERR_ALIGN."""
    return (b.or_bucket * 1)(b.or_bucket(grads=(1 << 30) + 4, masks=1 << 31, out=1 << 32, shard_len=4096))


def _status(*args, **kw):
    with pytest.raises(b.OptiReduceError) as e:
        b.or_fused_path_batched(*args, **kw)
    return e.value.status


def test_descriptor_arrays_in_every_form_that_ctypes_casts(arr):
    for form in (arr, C.pointer(arr[0]), C.pointer(arr), C.cast(arr, C.POINTER(b.or_bucket)), C.c_void_p(C.addressof(arr)),
                 C.addressof(arr), C.byref(arr), bytes(arr)):
        assert _status(form, 1, 2, 12, 0, None, 1) == BAD_ALIGN, form
    assert _status(None, 1, 2, 12, 0, None, 1) == 1                       # OR_ERR_NULL
    for form in (arr[0], bytearray(arr), np.frombuffer(bytes(arr), dtype=np.uint8), [1], 1.5):
        with pytest.raises(C.ArgumentError):
            b.or_fused_path_batched(form, 1, 2, 12, 0, None, 1)
