"""Softmaxes of a stack that share a launch though their shapes, strides and places differ: every part has the bits it has alone."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W

from . import harness as H
from . import launch_plan as L

pytestmark = pytest.mark.gpu
DEV = "cuda"
# (rows, columns, elements into a line): every lane count of the short rows; the workgroup-wide kernels; the long ones
STACKS = {
    "f32": [[(34900, 64, 0), (22990, 97, 1), (17200, 130, 0), (7450, 300, 3), (2230, 1000, 0), (1100, 2049, 0), (750, 3000, 5), (450, 5000, 0)],
            [(375, 6000, 0), (300, 8000, 1), (185, 12300, 0), (2000, 6000, 0)], [(190, 12000, 0), (160, 15000, 1), (140, 16384, 0)],
            [(140, 16400, 1), (60, 20011, 0), (700, 17000, 2), (9, 40003, 0)], [(5, 60011, 0), (300, 65536, 0), (300, 100003, 1)],
            [(6, 60011, 0), (18, 131041, 1), (300, 100003, 0)]],
    "bf16": [[(69700, 64, 0), (46000, 97, 1), (14900, 300, 0), (4500, 1000, 3), (6000, 751, 0), (2200, 2049, 0), (1500, 3000, 0), (600, 8001, 5)],
             [(400, 12000, 1), (300, 15000, 0), (250, 20011, 5)], [(190, 24000, 0), (200, 24064, 3)],
             [(64, 30205, 0), (700, 33000, 1), (9, 60011, 0)], [(20, 80003, 0), (300, 131072, 1), (5, 163000, 0)]],
}


def desc(dt, masked):
    if not masked:
        return W.get_program(f"softmax_{dt}")
    return W._p(f"masked_softmax_{dt}", [("z", dt), ("mask", dt)], [("s", "add", ["z", "mask"], {}), ("p", "softmax", ["s"], {})], [("p", dt)])


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_unlike_parts(dt, masked):
    ctx = B.Context(torch.cuda.current_device())
    ctx.set_limits(16, 2)           # (one interpreter variant for all parts)
    stream = torch.cuda.current_stream().cuda_stream
    for shapes in STACKS[dt]:
        print(f"[case] stack of softmaxes {dt} {shapes}{', masked' if masked else ''}", flush=True)
        codes, ins, outs, alone = [], [], [], []
        for k, (rows, cols, at) in enumerate(shapes):
            x = [gen.randn((rows, cols), 90 + k, DEV, dt, std=3.0)]
            if masked:
                x.append(gen.randn((1, cols) if k % 2 else (rows, cols), 120 + k, DEV, dt))
            room = torch.full((rows * cols + 256,), 7.0, dtype=x[0].dtype, device=DEV)
            y = room[64 + at: 64 + at + rows * cols].view(rows, cols)
            codes.append(B.encode_for(ctx, H.program(desc(dt, masked)), x, [y]))
            B.run_on(ctx, codes[-1], x + [y])
            torch.cuda.synchronize()
            alone.append(y.clone())
            want = torch.softmax((x[0][:3].float() + x[1][:3].float() if masked else x[0][:3]).double(), -1)
            rel = 4e-5 if dt == "f32" else 2.0 ** -8 + 4e-5      # (as in the tests of the kernels alone)
            assert bool(((y[:3].double() - want).abs() <= rel * want + 1e-37).all())
            room.fill_(7.0)
            ins.append(x)
            outs.append((room, y, at))
        ptrs = [t.data_ptr() for x, (_, y, _) in zip(ins, outs) for t in x + [y]]
        stack = B.dvm_stack(codes)
        plan = L.launches(stack, [ptrs])
        assert sum(l.n_segments for l in plan) == len(shapes) and all(l.kind != L.INTERPRETER for l in plan)
        (mixed,) = [l for l in plan if l.mixed]
        assert mixed.n_segments >= len(shapes) - 1      # (the largest may fill the chip and go alone)
        table = torch.empty(2 * len(ptrs), dtype=torch.int64, device=DEV)
        for batched in (False, True):
            for room, _, _ in outs:
                room.fill_(7.0)
            if batched:         # (a second set that writes the first set's results again)
                B.dvm_run_batched(ctx, stack, [ptrs, ptrs], table.data_ptr(), table.numel() * 8, stream)
            else:
                B.dvm_run(ctx, stack, ptrs, stream)
            torch.cuda.synchronize()
            for (room, y, at), ref in zip(outs, alone):
                assert torch.equal(y, ref), (batched, tuple(y.shape))
                assert bool((room[: 64 + at] == 7.0).all()) and bool((room[64 + at + y.numel():] == 7.0).all())


def test_two_threads():
    """Two threads launch rows of different lengths through one kernel, on a stream each."""
    import threading
    ctx = H.gpu_ctx()
    errors = []

    def work(cols, seed):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                x = gen.randn((300, cols), seed, DEV, "f32", std=3.0)
                code = B.encode_for(ctx, B.Program(W.get_program("softmax_f32")), [x])
                y, ref = torch.empty_like(x), torch.softmax(x.double(), -1)
                for _ in range(20):
                    y.fill_(7.0)
                    B.run_on(ctx, code, [x, y], stream.cuda_stream)
                    assert bool(((y.double() - ref).abs() <= 2e-5 * ref + 1e-37).all())
        except BaseException as e:
            errors.append(e)
    print("[case] two threads, fp32 [300, 85011] and [300, 114000]", flush=True)
    threads = [threading.Thread(target=work, args=a) for a in ((85011, 140), (114000, 141))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
