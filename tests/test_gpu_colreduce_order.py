"""Plain reductions along the penultimate axis: a launch of its own (dvm_colreduce) adds the rows in the order of the bytecode, the
one the interpreter takes for the same bytecode in a batched launch or a stack, whatever the context it runs under."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads.programs import _p, single_op_program

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
# several partial results per wave and one; fewer rows than partial results; ragged widths; many units
SHAPES = [(1, 4096, 512), (2, 300, 4096), (6, 1109, 2048), (1, 9238, 260), (1, 40, 515), (3, 5, 9), (161, 117, 1024), (256, 64, 513), (1, 16, 12)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_alone_batched_and_stacked(shape, dt):
    stream = torch.cuda.current_stream().cuda_stream
    for op in ("csum", "cmax"):
        print(f"[case] {op} {dt} {shape} alone, under another context, batched, stacked", flush=True)
        desc = _p(f"order_{op}", [("x", dt)], [("s", op, ["x"], {})], [("s", "f32")])
        ctx, other = B.Context(torch.cuda.current_device()), B.Context(torch.cuda.current_device())
        other.set_planner(37, 0)
        xs = [gen.randn(shape, 21 + i, DEV, dt) for i in range(3)]
        for c in (ctx, other):
            code = B.encode_for(c, H.program(desc), [xs[0]])
            new = [torch.full((shape[0], 1, shape[2]), -7.0, device=DEV) for _ in range(9)]
            alone, batch, stack = new[:3], new[3:6], new[6:]
            for x, s in zip(xs, alone):
                B.run_on(ctx, code, [x, s])
            again = torch.empty_like(alone[0])
            B.run_on(other, code, [xs[0], again])
            table = torch.empty(6, dtype=torch.int64, device=DEV)
            B.dvm_run_batched(ctx, code, [[x.data_ptr(), s.data_ptr()] for x, s in zip(xs, batch)], table.data_ptr(), 48, stream)
            B.dvm_run(ctx, B.dvm_stack([code] * 3), [t.data_ptr() for x, s in zip(xs, stack) for t in (x, s)], stream)
            torch.cuda.synchronize()
            assert torch.equal(again, alone[0])
            for k in range(3):
                assert torch.equal(batch[k], alone[k]) and torch.equal(stack[k], alone[k]), (op, k)


def test_beside_another_program():
    print("[case] a column sum stacked with a softmax", flush=True)
    ctx = B.Context(torch.cuda.current_device())
    ctx.set_limits(8, 2)
    x, z = gen.randn((2, 700, 1030), 25, DEV), gen.randn((300, 1000), 26, DEV)
    s, p = H.program(_p("order_csum", [("x", "f32")], [("s", "csum", ["x"], {})], [("s", "f32")])), H.program(single_op_program("softmax", 1))
    codes = [B.encode_for(ctx, s, [x]), B.encode_for(ctx, p, [z])]
    alone, both = [[torch.full((2, 1, 1030), -7.0, device=DEV), torch.full_like(z, -7.0)] for _ in range(2)]
    B.run_on(ctx, codes[0], [x, alone[0]])
    B.run_on(ctx, codes[1], [z, alone[1]])
    B.dvm_run(ctx, B.dvm_stack(codes), [t.data_ptr() for t in (x, both[0], z, both[1])], torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(both[0], alone[0]) and torch.equal(both[1], alone[1])
