"""The kernel launches of a run as the library plans them (csrc/dvm_internal.h: dvm_launch_plan), without a device."""
from __future__ import annotations

import ctypes as C
from typing import List, Sequence

from paper_2603_24239_amd import binding as B

INTERPRETER, SOFTMAX, SOFTMAX_LONG, SOFTMAX_EXACT, ROTARY = range(5)


class Launch(C.Structure):
    _fields_ = [(n, C.c_uint32) for n in ("kind", "first_segment", "n_segments", "grid", "block", "lanes", "slots", "mixed", "stream")]


def launches(code: B.Bytecode, sets: Sequence[Sequence[int]], n_cu: int = 256) -> List[Launch]:
    """`sets`: addresses of the tensors, set after set (they need not exist)."""
    fn = B.load().dvm_launch_plan
    fn.argtypes = [C.c_void_p, C.c_size_t, C.POINTER(C.c_void_p), C.c_int, C.c_int, C.POINTER(Launch), C.c_int, C.POINTER(C.c_int)]
    flat = [p for s in sets for p in s]
    out, n = (Launch * 64)(), C.c_int()
    status = fn(code.ptr, len(code), (C.c_void_p * len(flat))(*flat), len(sets), n_cu, out, 64, n)
    if status != 0:
        raise B.DvmError(status, "dvm_launch_plan")
    return list(out[: n.value])
