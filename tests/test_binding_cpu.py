"""The calls of the binding that a launch goes through, in the extension module and through ctypes: the argument forms that they take, and
what they refuse."""
from __future__ import annotations

import ctypes as C
import glob
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2603_24239_amd import binding as B
from paper_2603_24239_amd import marshal_ctypes
from workloads import programs as W


@pytest.fixture(params=["module", "ctypes"])
def ctx(request, monkeypatch):
    c = B.Context(-1)
    c.set_planner(256)
    if request.param == "module":
        assert B._dvm.__name__.endswith("._dvm")
    else:
        marshal_ctypes.bind(B.load())
        monkeypatch.setattr(B, "_dvm", marshal_ctypes)
    return c


@pytest.mark.parametrize("shape,offset,dt", [((4, 1000), 0, "f32"), ((7,), 3, "f32"), ((3, 5, 64), 1, "bf16"), ((0, 8), 0, "f32")])
def test_tensors_and_shapes_encode_alike(ctx, shape, offset, dt):
    n = int(np.prod(shape))
    t = torch.zeros(n + 8, dtype=torch.float32 if dt == "f32" else torch.bfloat16)[offset: offset + n].view(shape)
    prog = B.Program(W.single_op_program("add", 2, dt))
    a = B.encode_for(ctx, prog, [t, t])
    b = B.dvm_encode(ctx, prog, [B.shape_of_tensor(t)] * 2)
    assert a.raw == b.raw and list(a.out_shapes) == list(b.out_shapes) == [tuple(shape)]
    assert a.needs_workspace() is False and B.encode_for(ctx, prog, iter([t, t]), iter([t])).info().n_tensors == 3


def test_refusals(ctx):
    prog = B.Program(W.single_op_program("abs", 1, "f32"))
    code = B.encode_for(ctx, prog, [torch.zeros(16)])
    with pytest.raises(B.DvmError, match=r"\(-3\)"):
        B.encode_for(ctx, prog, [torch.zeros((1,) * 7)])
    with pytest.raises(B.DvmError, match="dvm_encode"):
        B.encode_for(ctx, prog, [torch.zeros(3)] * 40)
    with pytest.raises(B.DvmError, match="dvm_encode"):
        B.encode_for(ctx, prog, [torch.zeros(3)], [])
    with pytest.raises(TypeError):
        B.dvm_encode(ctx, prog, [b"no shape"])
    for ptrs in ([0, None], [C.c_void_p(64), np.int64(64)], [64] * 40, ()):      # (a context without a device launches nothing)
        with pytest.raises(B.DvmError, match="dvm_run"):
            B.dvm_run(ctx, code, ptrs)
    for sets in ([[64, 64]], [(np.uint64(64), None)] * 3):
        with pytest.raises(B.DvmError, match="dvm_run_batched"):
            B.dvm_run_batched(ctx, code, sets, 64, 4096)
    with pytest.raises(AssertionError):
        B.dvm_run_batched(ctx, code, [[64, 64], [64]], 64, 4096)
    with pytest.raises(IndexError):
        B.dvm_run_batched(ctx, code, [], 64, 4096)
    with pytest.raises(B.DvmError, match="dvm_stack"):
        B.dvm_stack([])
    assert B.dvm_stack([code, code]).info().n_segments == 2


def test_buffers_are_checked(ctx):
    code = B.encode_for(ctx, B.Program(W.single_op_program("abs", 1, "f32")), [torch.zeros(16)])
    whole = torch.zeros(32)
    B.check_buffers(code, [whole[:16], whole[16:]])
    with pytest.raises(B.DvmError, match="tensor 1: bytecode touches 64 bytes, storage holds 60"):
        B.check_buffers(code, [whole, whole[17:]])
    with pytest.raises(B.DvmError, match="tensor 0: bytecode touches 64 bytes, storage holds 0"):
        B.check_buffers(code, (whole[:0], whole))


class Yields:
    """A sequence that yields fewer addresses than its length says."""

    def __init__(self, at):
        self.at = at

    def __len__(self):
        return len(self.at) + 1

    def __getitem__(self, i):
        return self.at[i]

    def __iter__(self):
        return iter(self.at)


def test_sets_are_iterables_of_addresses(ctx):
    code = B.encode_for(ctx, B.Program(W.single_op_program("abs", 1, "f32")), [torch.zeros(16)])
    for sets in ([[64, 64], iter([64, 64])], [(64, 64), (p for p in (64, None))], ([64, 64], {64: 0, 128: 0})):
        with pytest.raises(B.DvmError, match="dvm_run_batched"):        # (a context without a device launches nothing)
            B.dvm_run_batched(ctx, code, sets, 64, 4096)
    for sets in ([[64, 64], iter([64])], [[64, 64], (p for p in range(64, 67))], [[64, 64], Yields([64])]):
        with pytest.raises(AssertionError):
            B.dvm_run_batched(ctx, code, sets, 64, 4096)
    with pytest.raises(TypeError):
        B.dvm_run_batched(ctx, code, [iter([64, 64])], 64, 4096)


@pytest.mark.parametrize("built", ["*.so", "libdvm.so"])
def test_a_build_in_the_process_that_uses_it(tmp_path, built):
    """A clean tree's build imports the package, compiles, and loads what it compiled, all in one process; without the extension module too."""
    here = os.path.dirname(B.__file__)
    pkg = tmp_path / os.path.basename(here)
    pkg.mkdir()
    for f in glob.glob(os.path.join(here, "*.py")):
        shutil.copy(f, pkg)
    script = ("import glob, shutil\n"
              "from paper_2603_24239_amd import binding as B\n"
              f"for f in glob.glob({os.path.join(here, built)!r}): shutil.copy(f, {str(pkg)!r})\n"
              "B.load()\n"
              f"assert B.__file__.startswith({str(pkg)!r})\n"
              f"assert B._dvm.__name__.endswith({'._dvm' if built == '*.so' else '.marshal_ctypes'!r})\n"
              "assert B.Context(-1).device == -1\n")
    r = subprocess.run([sys.executable, "-c", script], cwd=tmp_path, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
