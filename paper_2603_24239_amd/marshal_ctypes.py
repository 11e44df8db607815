"""The calls of the extension module (csrc/dvm_py.c) through ctypes, with the same arguments and results: for an installation whose build found no
headers of the Python interpreter.  4 to 12 us of host time a call instead of 1 to 3."""
from __future__ import annotations

import ctypes as C
import struct

MAX_RANK, MAX_TENSORS, ENC_CAP = 6, 32, 8192
E_ARGS, E_LIMIT = -1, -10
_SHAPE = struct.Struct(f"=ii{MAX_RANK}q{MAX_RANK}q")        # a whole dvm_shape
_PAD = [(0,) * (MAX_RANK - r) for r in range(MAX_RANK + 1)]
_lib = None


def bind(lib) -> None:
    global _lib
    _lib = lib


def _shapes(seq, with_shapes):
    """(count, buffer of dvm_shapes); the buffer is None where a rank exceeds the limit."""
    seq = list(seq)
    buf = C.create_string_buffer(max(len(seq), 1) * _SHAPE.size)
    for k, t in enumerate(seq[:MAX_TENSORS]):
        if with_shapes:
            raw = memoryview(t).cast("B")
            if len(raw) != _SHAPE.size:
                raise TypeError("a dvm_shape")
            buf[k * _SHAPE.size: (k + 1) * _SHAPE.size] = raw.tobytes()
            continue
        dims, strides, p = t.shape, t.stride(), t.data_ptr()
        if len(dims) > MAX_RANK:
            return len(seq), None
        pad = _PAD[len(dims)]
        _SHAPE.pack_into(buf, k * _SHAPE.size, len(dims), p & -p if p & 15 else 16, *dims, *pad, *strides, *pad)
    return len(seq), buf


def encode(ctx, prog, inputs, outputs, n_out, with_shapes):
    n_in, ins = _shapes(inputs, with_shapes)
    n_lay, lay = (n_out, b"") if outputs is None or ins is None else _shapes(outputs, with_shapes)
    if ins is None or lay is None:
        return None
    if n_in > MAX_TENSORS or n_lay > MAX_TENSORS or n_out > MAX_TENSORS or n_lay < n_out:
        return E_ARGS
    buf, outs, n = C.create_string_buffer(ENC_CAP), C.create_string_buffer(MAX_TENSORS * _SHAPE.size), C.c_size_t()
    shapes_at = _lib.dvm_encode.argtypes[2]
    st = _lib.dvm_encode(ctx, prog, C.cast(ins, shapes_at), n_in, None if outputs is None else C.cast(lay, shapes_at), buf, ENC_CAP, n, C.cast(outs, shapes_at))
    if st != 0:
        return st
    dims = [_SHAPE.unpack_from(outs, k * _SHAPE.size) for k in range(n_out)]
    return buf.raw[: n.value], [v[2: 2 + v[0]] for v in dims]


def _addresses(seq):
    out = []
    for p in seq:
        p = p.value if isinstance(p, C.c_void_p) else p
        out.append(0 if p is None else p.__index__())
    return out


def run(ctx, code, addresses, stream):
    p = _addresses(addresses)
    if len(p) > MAX_TENSORS:
        return E_ARGS
    return _lib.dvm_run(ctx, code, len(code), (C.c_void_p * max(len(p), 1))(*p), len(p), stream)


def run_batched(ctx, code, sets, table, table_bytes, stream):
    sets = [_addresses(s) for s in sets]
    n = len(sets[0]) if sets else 0
    if any(len(s) != n for s in sets):
        return None
    flat = (C.c_void_p * max(n * len(sets), 1))(*[p for s in sets for p in s])
    return _lib.dvm_run_batched(ctx, code, len(code), flat, n, len(sets), table, table_bytes, stream)


def stack(codes, spatial):
    if len(codes) > MAX_TENSORS:            # (every part has a tensor)
        return E_LIMIT
    ptrs = (C.c_void_p * max(len(codes), 1))(*[C.cast(C.c_char_p(c), C.c_void_p) for c in codes])
    lens = (C.c_size_t * max(len(codes), 1))(*[len(c) for c in codes])
    buf, n = C.create_string_buffer(ENC_CAP), C.c_size_t()
    st = (_lib.dvm_stack_spatial if spatial else _lib.dvm_stack)(ptrs, lens, len(codes), buf, ENC_CAP, n)
    return st if st != 0 else buf.raw[: n.value]


def check(code, tensors):
    tensors = list(tensors)
    need = (C.c_int64 * MAX_TENSORS)()
    st = E_ARGS if len(tensors) > MAX_TENSORS else _lib.dvm_code_min_bytes(code, len(code), need, len(tensors))
    if st != 0:
        return st
    for i, t in enumerate(tensors):
        have = t.untyped_storage().nbytes()
        offset = t.storage_offset()
        if offset != 0:
            have -= offset * t.element_size()
        numel = t.numel()
        if need[i] > have or (numel == 0 and need[i] > 0):
            return i, need[i], have if numel else 0
    return None


def needs_workspace(code):
    info = _lib.dvm_code_info_get.argtypes[2]._type_()
    st, kind = _lib.dvm_code_info_get(code, len(code), info), C.c_int()
    if st == 0 and info.n_tensors > 0:
        st = _lib.dvm_code_tensor(code, len(code), info.n_tensors - 1, None, kind, None, None)
    return st if st != 0 else kind.value == 2
