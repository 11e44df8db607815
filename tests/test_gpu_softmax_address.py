"""The bits of a softmax do not depend on addresses: rows of whole 128-byte lines in an output that starts inside one, alone and in a batch with others."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
# (the shift takes a slot more, or its kernel has none more and the rows stay where they are)
COLS = {"f32": [192, 448, 2048, 16384, 32768, 131072], "bf16": [448, 1984, 16384, 65536, 163840]}


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_outputs_on_and_off_a_line(dt):
    es = 4 if dt == "f32" else 2
    ctx = H.gpu_ctx()
    prog = H.program(W.get_program(f"softmax_{dt}"))
    stream = torch.cuda.current_stream().cuda_stream
    for cols in COLS[dt]:
        rows = -(-(17 << 20) // (2 * es * cols))
        xs = [gen.randn((rows, cols), 80 + k, DEV, dt, std=3.0) for k in range(3)]
        code = B.dvm_encode(ctx, prog, [B.make_shape((rows, cols), align_bytes=es)], [B.make_shape((rows, cols), align_bytes=es)])

        def room(at):
            r = torch.full((rows * cols + 256,), 7.0, dtype=xs[0].dtype, device=DEV)
            return r, r[64 + at: 64 + at + rows * cols].view(rows, cols)
        refs = [room(0) for _ in xs]
        assert refs[0][1].data_ptr() % 128 == 0
        for x, (_, y) in zip(xs, refs):
            B.run_on(ctx, code, [x, y])
        want = torch.softmax(xs[0][:5].double(), -1)
        assert bool(((refs[0][1][:5].double() - want).abs() <= (2e-5 if dt == "f32" else 2.0 ** -8 + 2e-5) * want + 1e-37).all())
        for at in (1, 16 // es, 124 // es):
            print(f"[case] softmax {dt} [{rows}, {cols}], output {at} elements into a line, alone and in a batch of three", flush=True)
            whole, y = room(at)
            B.run_on(ctx, code, [xs[0], y])
            torch.cuda.synchronize()
            assert torch.equal(y, refs[0][1]), (cols, at)
            outs = [room(0), room(at), room(0)]
            table = torch.empty(6, dtype=torch.int64, device=DEV)
            B.dvm_run_batched(ctx, code, [[x.data_ptr(), o.data_ptr()] for x, (_, o) in zip(xs, outs)], table.data_ptr(), 48, stream)
            torch.cuda.synchronize()
            for (_, o), (_, r) in zip(outs, refs):
                assert torch.equal(o, r), (cols, at)
            for r, o in outs + [(whole, y)]:
                first = (o.data_ptr() - r.data_ptr()) // es
                assert bool((r[:first] == 7.0).all()) and bool((r[first + rows * cols:] == 7.0).all())
