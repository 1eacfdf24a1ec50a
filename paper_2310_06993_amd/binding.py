"""Thin binding of liboptireduce_hip.so: argument marshalling only (ctypes; natively where kernels are enqueued).

Every function has the name and argument order of its C entry point in include/optireduce.h and
takes torch tensors that already live on the GPU (torch is used for device memory and streams,
nothing else).  A non-zero status raises OptiReduceError.  There is no CPU fallback: if the
library or the native marshalling module is not built, importing this module raises.
"""
from __future__ import annotations

import ctypes as C
import os

import torch  # noqa: F401  (its libraries have to be loaded before the native module)

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "liboptireduce_hip.so")
if not os.path.exists(_LIB_PATH):
    raise ImportError(
        "liboptireduce_hip.so is not built (%s); run `python -m paper_2310_06993_amd.build`" % _LIB_PATH)
lib = C.CDLL(_LIB_PATH)

from . import _calls  # noqa: E402

_u64, _int, _p, _sz = C.c_uint64, C.c_int, C.c_void_p, C.c_size_t

OR_OK = 0
OR_MIN_LOG2, OR_MAX_LOG2, OR_MAX_WORKERS = 5, 16, 255

_SIGS = {
    "or_padded_len": (_u64, [_u64, _int]),
    "or_workspace_bytes": (_sz, [_u64, _int]),
    "or_status_string": (C.c_char_p, [_int]),
    "or_version": (_int, []),
    "or_last_hip_error": (_int, []),
    "or_time_next_call": (_int, [_p, _p]),
    "or_rht_encode": (_int, [_p, _u64, _int, _u64, _p, _p]),
    "or_rht_encode_at": (_int, [_p, _u64, _int, _u64, _u64, _p, _p]),
    "or_rht_encode_bf16": (_int, [_p, _u64, _int, _u64, _u64, _p, _p]),
    "or_masked_reduce": (_int, [_p, _p, _int, _u64, _p, _p, _p]),
    "or_masked_reduce_bf16": (_int, [_p, _p, _int, _u64, _p, _p, _p]),
    "or_rht_decode": (_int, [_p, _u64, _int, _u64, _p, _p]),
    "or_rht_decode_at": (_int, [_p, _u64, _int, _u64, _u64, _p, _p]),
    "or_rht_decode_bf16": (_int, [_p, _u64, _int, _u64, _u64, _p, _p]),
    "or_finalize_decode": (_int, [_p, _p, _u64, _int, _u64, _u64, _p, _p]),
    "or_finalize_decode_bf16": (_int, [_p, _p, _u64, _int, _u64, _u64, _p, _p]),
    "or_reduce_decode": (_int, [_p, _p, _int, _u64, _int, _u64, _u64, _p, _p, _p, _sz, _p]),
    "or_reduce_decode_bf16": (_int, [_p, _p, _int, _u64, _int, _u64, _u64, _p, _p, _p, _sz, _p]),
    "or_fused_path": (_int, [_p, _p, _int, _u64, _int, _u64, _u64, _p, _p, _p, _sz, _p]),
    "or_fused_path_bf16": (_int, [_p, _p, _int, _u64, _int, _u64, _u64, _p, _p, _p, _sz, _p]),
    "or_fused_path_bf16_static": (_int, [_p, _p, _int, _u64, _int, _u64, _u64, _p, _p, _p]),
    "or_fused_path_batched": (_int, [_p, _int, _int, _int, _int, _p, _sz, _p]),
    "or_fused_path_batched_monitored": (_int, [_p, _int, _int, _int, _int, _p, _p, _sz, _p]),
    "or_reduce_decode_batched": (_int, [_p, _int, _int, _int, _int, _p, _p, _sz, _p]),
    "or_masked_reduce_batched": (_int, [_p, _int, _int, _int, _p]),
    "or_finalize_decode_batched": (_int, [_p, _int, _int, _int, _p]),
    "or_finalize": (_int, [_p, _p, _u64, _p, _p]),
    "or_finalize_bf16": (_int, [_p, _p, _u64, _p, _p]),
    "or_received_total": (_int, [_p, _u64, _p, _p]),
    "or_loss_decision": (_int, [_u64, _int, _u64, _p, _int, _p, _p, _p]),
    "or_rht_decode_masked": (_int, [_p, _p, _u64, _int, _u64, _u64, _p, _p]),
    "or_rht_decode_masked_bf16": (_int, [_p, _p, _u64, _int, _u64, _u64, _p, _p]),
    "or_masked_reduce_pairs": (_int, [_p, _p, _p, _int, _u64, _p, _p, _p]),
}


OR_ACT_APPLY, OR_ACT_SKIP, OR_ACT_HALT = 0, 1, 2
OR_DEFAULT_TRANSFORM_ON_LOSS = 0.02


class or_loss_policy(C.Structure):
    _fields_ = [("transform_on_loss", C.c_double), ("skip_loss", C.c_double), ("halt_loss", C.c_double)]


class or_bucket(C.Structure):
    _fields_ = [("grads", _p), ("masks", _p), ("out", _p), ("count_out", _p),
                ("shard_len", _u64), ("seed", _u64), ("base_index", _u64)]


class or_stage_bucket(C.Structure):
    _fields_ = [("shards", _p), ("masks", _p), ("sum", _p), ("count", _p), ("out", _p),
                ("shard_len", _u64), ("seed", _u64), ("base_index", _u64)]


for _name, (_res, _args) in _SIGS.items():
    _f = getattr(lib, _name)
    _f.restype, _f.argtypes = _res, _args


class OptiReduceError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__("%s: status %d (%s)" % (where, status, lib.or_status_string(status).decode()))


def _ptr(t):
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("liboptireduce_hip takes device tensors")
    if not t.is_contiguous():
        raise ValueError("tensor must be contiguous")
    return t.data_ptr()


def _check(status, where):
    if status != OR_OK:
        raise OptiReduceError(status, where)


def or_padded_len(n: int, block_log2: int) -> int:
    return int(lib.or_padded_len(n, block_log2))


def or_workspace_bytes(shard_len: int, block_log2: int) -> int:
    return int(lib.or_workspace_bytes(shard_len, block_log2))


def or_version() -> int:
    return int(lib.or_version())


def or_time_next_call(start_event, stop_event):
    """start_event / stop_event: raw hipEvent_t handles (ints) or None."""
    _check(lib.or_time_next_call(start_event, stop_event), "or_time_next_call")


# The entry points that enqueue kernels, marshalled natively (csrc/calls.cpp): same names and argument order as the C
# ones, device pointers are tensors or None, a workspace carries its own size, `count_out`, `workspace`, `totals` (of
# or_reduce_decode_batched) and `stream` may be left out.  `stream`: None (the current stream), a torch stream or a raw
# handle.  Descriptor arrays are those of make_buckets / make_stage_buckets; `totals` an int64 device tensor of n_buckets
# entries (or_received_total: one entry).
from ._calls import (  # noqa: E402
    or_finalize, or_finalize_bf16, or_finalize_decode, or_finalize_decode_batched, or_finalize_decode_bf16, or_fused_path,
    or_fused_path_batched, or_fused_path_batched_monitored, or_fused_path_bf16, or_fused_path_bf16_static, or_masked_reduce,
    or_masked_reduce_batched, or_masked_reduce_bf16, or_masked_reduce_pairs, or_received_total, or_reduce_decode,
    or_reduce_decode_batched, or_reduce_decode_bf16, or_rht_decode, or_rht_decode_at, or_rht_decode_bf16,
    or_rht_decode_masked, or_rht_decode_masked_bf16, or_rht_encode, or_rht_encode_at, or_rht_encode_bf16)



def _integer(o, unsigned):
    """What ctypes makes of an argument that is no int: its own integer of the right type, or _as_parameter_."""
    kind = _u64 if unsigned else _int
    while not isinstance(o, kind) and hasattr(o, "_as_parameter_"):
        o = o._as_parameter_
    try:
        return o.value if isinstance(o, kind) else kind(o).value
    except TypeError as e:
        raise C.ArgumentError(str(e)) from None


def _extent(o, sized):
    return _ptr(o), o.numel() * o.element_size() if sized else 0


_calls.bind({name: C.cast(getattr(lib, name), _p).value for name in _SIGS}, _check, C.Array, lambda o: C.cast(o, _p).value,
            _integer, _extent)

OR_STATIC_MAX_SHARD_LEN = 4194304


def make_buckets(items):
    """items: iterable of (grads, masks, out, count_out_or_None, shard_len, seed, base_index) with device
    tensors -> a host array of or_bucket that or_fused_path_batched can take (reusable across calls)."""
    items = list(items)
    arr = (or_bucket * len(items))()
    for j, (g, m, o, c, L, seed, base) in enumerate(items):
        arr[j] = or_bucket(_ptr(g), _ptr(m), _ptr(o), _ptr(c), L, seed, base)
    return arr


def make_stage_buckets(items):
    """items: iterable of (shards, masks, sum, count, out, shard_len, seed, base_index) with device tensors
    (or None where the call ignores the field) -> a host array of or_stage_bucket."""
    items = list(items)
    arr = (or_stage_bucket * len(items))()
    for j, (sh, m, t, c, o, L, seed, base) in enumerate(items):
        arr[j] = or_stage_bucket(_ptr(sh), _ptr(m), _ptr(t), _ptr(c), _ptr(o), L, seed, base)
    return arr


def or_loss_decision(received_total, N, shard_len, policy, prev_transform_on):
    """Host arithmetic only.  policy: an or_loss_policy.  Returns (action, transform_on, loss)."""
    act, ton, loss = C.c_int(), C.c_int(), C.c_double()
    _check(lib.or_loss_decision(int(received_total), N, shard_len, C.byref(policy), int(bool(prev_transform_on)),
                                C.byref(act), C.byref(ton), C.byref(loss)), "or_loss_decision")
    return act.value, ton.value, loss.value
