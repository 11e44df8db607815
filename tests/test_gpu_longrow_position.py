"""Rows longer than a tile: equal rows give equal bits wherever they stand -- in programs of two, three and four passes, with more rows
than workgroups, under both assignments, and as parts of a batched launch or a stack."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W
from workloads.programs import _p, single_op_program

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
ROWS, COLS, KINDS = 2600, 60011, 13     # (1024 workgroups at most: every one runs two rows or more; thirteen different rows in turn)


def programs():
    four = _p("four", [("x", "f32")], [("m", "mean", ["x"], {}), ("d", "sub", ["x", "m"], {}), ("v", "meansq", ["d"], {}), ("q", "square", ["d"], {}), ("c", "mul", ["q", "v"], {}),
                                       ("s", "sum", ["c"], {}), ("y", "mul", ["d", "s"], {})], [("y", "f32")])
    return {"softmax": single_op_program("softmax", 1, "f32"), "layernorm": W.get_program("layernorm_f32"), "four": four}


def context(assignment="auto"):
    c = B.Context(torch.cuda.current_device())
    c.set_assignment(assignment)
    return c


def inputs(name, rows):
    x = gen.randn((KINDS, COLS), 71, DEV).repeat(rows // KINDS, 1)
    return {"a0": x} if name == "softmax" else {"x": x} if name == "four" else \
        {"x": x, "gamma": gen.randn((COLS,), 72, DEV, mean=1.0, std=0.1), "beta": gen.randn((COLS,), 73, DEV, std=0.1)}


@pytest.mark.parametrize("assignment", ["interleaved", "blocked"])
@pytest.mark.parametrize("name", ["softmax", "layernorm", "four"])
def test_equal_rows_give_equal_bits(name, assignment):
    print(f"[case] {name} [{ROWS}, {COLS}] of 13 rows in turn, {assignment}", flush=True)
    desc = programs()[name]
    one, _ = H.run_vm(desc, inputs(name, KINDS), ctx=context())
    many, code = H.run_vm(desc, inputs(name, ROWS), ctx=context(assignment))
    assert code.info().grid < ROWS
    y = many["y"]
    assert torch.equal(y.view(-1, KINDS, COLS), one["y"].expand(ROWS // KINDS, KINDS, COLS))


def test_long_rows_in_a_batch_and_in_a_stack():
    n, rows = 5, 300
    for name, desc in programs().items():
        print(f"[case] {name}: {n} sets and {n} parts of [{rows}, {COLS}]", flush=True)
        ctx = context()
        xs = [gen.randn((rows, COLS), 74 + i, DEV) for i in range(n)]
        rest = list(inputs(name, KINDS).values())[1:]
        code = B.encode_for(ctx, H.program(desc), [xs[0]] + rest)
        refs = [torch.empty_like(x) for x in xs]
        for x, y in zip(xs, refs):
            B.run_on(ctx, code, [x] + rest + [y])
        stream = torch.cuda.current_stream().cuda_stream
        outs = [torch.full_like(x, -7.0) for x in xs]
        sets = [[t.data_ptr() for t in [x] + rest + [y]] for x, y in zip(xs, outs)]
        table = torch.empty(n * len(sets[0]), dtype=torch.int64, device=DEV)
        B.dvm_run_batched(ctx, code, sets, table.data_ptr(), table.numel() * 8, stream)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, refs)), name
        outs = [torch.full_like(x, -7.0) for x in xs]
        B.dvm_run(ctx, B.dvm_stack([code] * n), [t.data_ptr() for x, y in zip(xs, outs) for t in [x] + rest + [y]], stream)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, refs)), name
