"""Softmaxes alike in all but their addresses share one launch in a stack: another shape and another
program between them, and every part has the bits it has alone."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads.programs import single_op_program

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def soft(dt):
    return single_op_program("softmax", 1, dt)


@pytest.mark.parametrize("dt,rows,cols,other", [("f32", 5, 60011, 6), ("bf16", 40, 17001, 41), ("bf16", 5600, 751, 5601)])
def test_alike_parts_share_a_launch(dt, rows, cols, other):
    ctx = B.Context(torch.cuda.current_device())
    add = single_op_program("add", 2, dt)
    parts = [(soft(dt), [gen.randn((rows, cols), 10 + i, DEV, dt)]) for i in range(11)]
    parts.insert(2, (soft(dt), [gen.randn((other, cols), 40, DEV, dt)]))
    parts.insert(4, (add, [gen.randn((64, 128), 41, DEV, dt), gen.randn((64, 128), 42, DEV, dt)]))
    codes = [B.encode_for(ctx, H.program(d), ins) for d, ins in parts]
    alone = [torch.empty_like(ins[0]) for _, ins in parts]
    for (_, ins), code, y in zip(parts, codes, alone):
        B.run_on(ctx, code, ins + [y])
    outs = [torch.full_like(y, -7.0) for y in alone]
    B.dvm_run(ctx, B.dvm_stack(codes), [t.data_ptr() for (_, ins), y in zip(parts, outs) for t in ins + [y]],
              torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for a, b in zip(outs, alone):
        assert torch.equal(a, b)
    want = torch.softmax(parts[0][1][0].double(), -1)
    # an argument of the exponential is below 2^4 and rounds by 2^-20 at most, each term of a lane's sum and of the tree over lanes by 2^-24: fewer
    # than 2^7 of them one after the other; bf16 rounds the result by 2^-9 of the next power of two
    tol = 2.0 ** -20 * 8 + 2.0 ** -17 + (2.0 ** -8 if dt == "bf16" else 0.0)
    assert bool(((outs[0].double() - want).abs() <= tol * want + 1e-30).all())
