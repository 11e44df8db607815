"""Rows that end inside a 16-byte chunk: the last chunk slides back over its neighbour.  Widths around a chunk, around a wave
and where the neighbour belongs to another wave, against the oracle; and programs that write their own input, which must give
the bits of the same program writing elsewhere."""
from __future__ import annotations

import pytest
import torch

from workloads import gen
from workloads.programs import _p, single_op_program

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
COLS = [3, 5, 9, 31, 65, 255, 513, 1027, 2049, 4099, 8195]


def norm_affine(dt):
    """Two reductions, two row-invariant operands (kept in LDS where the plan wants that) and one read again."""
    return _p("norm_affine", [("x", dt), ("r", dt), ("g", dt), ("b", dt), ("c", dt)],
              [("h", "add", ["x", "r"], {}), ("m", "mean", ["h"], {}), ("d", "sub", ["h", "m"], {}), ("v", "meansq", ["d"], {}),
               ("ve", "adds", ["v"], {"imm": 1e-5}), ("s", "rsqrt", ["ve"], {}), ("n", "mul", ["d", "s"], {}), ("ng", "mul", ["n", "g"], {}),
               ("nb", "add", ["ng", "b"], {}), ("nc", "add", ["nb", "c"], {}), ("t", "silu", ["nc"], {}), ("y", "add", ["t", "h"], {})],
              [("y", dt)])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("cols", COLS)
def test_widths(dt, cols):
    print(f"[case] ragged rows {dt} [37, {cols}]", flush=True)
    x = gen.randn((37, cols), 31, DEV, dt, std=3.0)
    x[3, cols - 1] = 40.0               # the maximum in the last element
    x[4, :] = -5.0
    x[5, 0] = float("nan")
    x[6, cols - 1] = float("inf")
    H.check_program(single_op_program("softmax", 1, dt), {"a0": x})
    H.check_program(single_op_program("rmin", 1, dt), {"a0": x})
    d = {"x": gen.randn((37, cols), 32, DEV, dt), "r": gen.randn((37, cols), 33, DEV, dt), "g": gen.randn((cols,), 34, DEV, dt, mean=1.0, std=0.1),
         "b": gen.randn((cols,), 35, DEV, dt, std=0.1), "c": gen.randn((cols,), 36, DEV, dt, std=0.1)}
    H.check_program(norm_affine(dt), d)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("cols", COLS + [20483])
def test_a_program_that_writes_its_input(dt, cols):
    print(f"[case] in place {dt} [37, {cols}]", flush=True)
    x = gen.randn((37, cols), 41, DEV, dt)
    # (early: stored before the row's maximum is taken; late: stored after it)
    early = _p("early", [("x", dt)], [("y", "adds", ["x"], {"imm": 100.0}), ("m", "rmax", ["x"], {})], [("y", dt), ("m", dt)])
    late = single_op_program("softmax", 1, dt)
    flat = single_op_program("gelu_tanh", 1, dt)
    for desc, name in ((early, "x"), (late, "a0"), (flat, "a0")):
        if desc is early and cols > 16384:
            continue
        ref, _ = H.run_vm(desc, {name: x})
        mine = x.clone()
        outs = {n: torch.empty_like(t) for n, t in ref.items()}
        outs["y"] = mine
        got, _ = H.run_vm(desc, {name: mine}, outputs=outs)
        for n in ref:
            assert torch.equal(got[n], ref[n]), (desc.name, n)
