"""Launches of many short segments and sets: every workgroup passes over those that hold none of its tiles.  Sets with fewer tiles
than workgroups and with more, empty segments, segments in blocked ranges beside round-robin ones; the bits of single launches."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("assignment", ["auto", "blocked"])
@pytest.mark.parametrize("rows,n_sets", [((0, 1, 3), 7), ((1, 40, 5), 64), ((700, 0, 2900), 3), ((5, 5, 5), 1)])
def test_sets_of_stacked_segments(rows, n_sets, assignment):
    print(f"[case] {n_sets} sets of segments with {rows} rows, {assignment}", flush=True)
    ctx = B.Context(torch.cuda.current_device())
    ctx.set_limits(32, 2)
    mixed = B.Context(torch.cuda.current_device())          # (the last segment as the assignment says, the others round-robin)
    mixed.set_limits(32, 2)
    mixed.set_assignment(assignment)
    prog = H.program(W.get_program("c2_rmsnorm"))
    parts = []
    for k, n in enumerate(rows):
        c = mixed if k + 1 == len(rows) else ctx
        w = gen.randn((1000,), 80 + k, DEV, "bf16", mean=1.0, std=0.1)
        x = gen.randn((n_sets, n, 1000), 90 + k, DEV, "bf16")
        parts.append((c, B.encode_for(c, prog, [x[0], w]), x, w, torch.full_like(x, -7.0)))
    stack = B.dvm_stack([p[1] for p in parts])
    sets = [[q for (_, _, x, w, y) in parts for q in (x[i].data_ptr() or w.data_ptr(), w.data_ptr(), y[i].data_ptr() or w.data_ptr())] for i in range(n_sets)]
    table = torch.empty(n_sets * len(sets[0]), dtype=torch.int64, device=DEV)
    stream = torch.cuda.current_stream().cuda_stream
    B.dvm_run_batched(ctx, stack, sets, table.data_ptr(), table.numel() * 8, stream)
    torch.cuda.synchronize()
    for c, code, x, w, y in parts:
        for i in range(n_sets):
            if x[i].numel() == 0:
                continue
            ref = torch.empty_like(y[i])
            B.run_on(c, code, [x[i], w, ref])
            assert torch.equal(y[i], ref), (tuple(x.shape), i)
