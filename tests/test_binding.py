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


class _Has:
    """_as_parameter_, as ctypes looks for it."""
    def __init__(self, value):
        self._as_parameter_ = value


class _TensorLike:
    """What the binding needs of a device tensor, without torch."""
    is_cuda = True

    def __init__(self, contiguous=True):
        self.contiguous = contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return (1 << 20) + 4

    def numel(self):
        return 3

    def element_size(self):
        return 2


def test_integers_in_every_form_that_ctypes_takes(arr):
    for one in (1, True, np.int64(1), C.c_int(1), _Has(1), _Has(C.c_int(1))):
        assert _status(arr, one, 2, 12, 0, None, 1) == BAD_ALIGN, one
    for bad in (1.0, None, "1", C.c_uint64(1), _Has(1.0), [1]):
        with pytest.raises(C.ArgumentError):
            b.or_fused_path_batched(arr, bad, 2, 12, 0, None, 1)
    for zero in (0, C.c_uint64(0), np.uint64(0), 1 << 64):
        b.or_rht_encode(None, zero, 10, -1, None, 1)                      # an empty vector
    with pytest.raises(C.ArgumentError):
        b.or_rht_encode(None, C.c_int(0), 10, 1, None, 1)


def test_tensors_and_what_looks_like_one():
    with pytest.raises(b.OptiReduceError) as e:
        b.or_rht_encode(_TensorLike(), 64, 10, 1, _TensorLike(), 1)
    assert e.value.status == BAD_ALIGN
    with pytest.raises(ValueError):
        b.or_rht_encode(_TensorLike(contiguous=False), 64, 10, 1, None, 1)
    with pytest.raises(AttributeError):
        b.or_rht_encode("x", 64, 10, 1, None, 1)
    # a workspace's size is taken from it: 6 bytes are too few
    one = (b.or_bucket * 1)(b.or_bucket(grads=1 << 30, masks=1 << 31, out=1 << 32, shard_len=1 << 16))
    with pytest.raises(b.OptiReduceError) as e:
        b.or_fused_path_batched(one, 1, 2, 16, 0, _TensorLike(), 1)
    assert e.value.status == 6


def test_an_error_of_the_runtime_leaves_nothing_held(arr):
    """No GPU: looking up the current stream raises after the descriptors were taken; they are let go."""
    import sys
    import torch
    if torch.cuda.is_available():
        pytest.skip("the stream is there")
    before = sys.getrefcount(arr)
    for _ in range(5):
        with pytest.raises(RuntimeError):
            b.or_fused_path_batched(arr, 1, 2, 12, 0, None)
    assert sys.getrefcount(arr) == before


def test_signatures_can_be_read():
    """Names, order and defaults of the arguments, as inspect and help() show them."""
    import inspect
    show = lambda f: str(inspect.signature(f))
    assert show(b.or_rht_encode) == "(grad, n, block_log2, seed, out, stream=None)"
    assert show(b.or_fused_path) == ("(grads, masks, N, shard_len, block_log2, seed, base_index, out, count_out=None, workspace=None, "
                                     "stream=None)")
    assert show(b.or_fused_path_batched_monitored) == "(buckets, n_buckets, N, block_log2, bf16, totals, workspace=None, stream=None)"
    assert show(b.or_reduce_decode_batched) == "(buckets, n_buckets, N, block_log2, bf16, totals=None, workspace=None, stream=None)"
    assert show(b.or_masked_reduce_pairs) == "(sums, counts, masks, G, shard_len, sum_out, count_out, stream=None)"
    for name in b._SIGS:
        if hasattr(b, name):
            assert inspect.signature(getattr(b, name)) is not None, name
