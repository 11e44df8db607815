"""Softmax of a sum of two tensors over rows that a workgroup holds: in every kernel for those, with full, broadcast and shared second tensors (the
last in blocks of rows), and written over either operand; against float64."""
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
INF = float("inf")
TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
# one width for each kernel: fp32 by 512 lanes in 16, 24 slots, by 1024 in 28, 33; bf16 by 512 in 8, 16, by 1024.  30205: the last chunk of a row of bf16,
# which slides back over columns of its neighbour, is the first of a wave for seven places in a line
COLS = {"f32": [20011, 40003, 100003, 114657, 131041], "bf16": [25089, 30205, 60011, 131071]}


def desc(dt):
    return W._p(f"masked_softmax_{dt}", [("z", dt), ("mask", dt)], [("s", "add", ["z", "mask"], {}), ("p", "softmax", ["s"], {})], [("p", dt)])


def check(got, z, mask, dt, what):
    """As for shorter rows: the exponential's argument carries a rounding of 2^-24 of itself, up to 1e-5 at the differences that matter, and the sum
    of the two tensors one more; bf16 rounds once more."""
    rel = 4e-5 if dt == "f32" else 2.0 ** -8 + 4e-5
    for k in range(0, got.shape[0], 64):
        m = mask if mask.shape[0] == 1 else mask[k: k + 64]
        ref = torch.softmax((z[k: k + 64].float() + m.float()).double(), dim=-1)
        err = (got[k: k + 64].double() - ref).abs()
        assert bool((torch.isnan(ref) == torch.isnan(got[k: k + 64])).all()), what
        assert bool((torch.isnan(ref) | (err <= rel * ref + 1e-37)).all()), (what, k)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_full_and_broadcast(dt):
    for cols in COLS[dt]:
        rows = 300              # (more than the workgroups of a launch)
        print(f"[case] masked softmax {dt} [{rows}, {cols}]", flush=True)
        z = gen.randn((rows, cols), 71, DEV, dt, std=3.0)
        full = gen.randn((rows, cols), 72, DEV, dt)
        full[1] = -INF
        full[2, cols // 3:] = -INF
        z[3, cols - 1] = float("nan")
        room = torch.full((rows * cols + 256,), 7.0, dtype=TORCH_DT[dt], device=DEV)
        for mask in (full, full[5:6]):
            for at in (0, 5):
                out = room[64 + at: 64 + at + rows * cols].view(rows, cols)
                _, code = H.run_vm(desc(dt), {"z": z, "mask": mask}, {"p": out})
                assert [l.kind for l in L.launches(code, [[z.data_ptr(), mask.data_ptr(), out.data_ptr()]])] == [L.SOFTMAX_LONG]
                check(out, z, mask, dt, (cols, mask.shape))
                assert bool((room[: 64 + at] == 7.0).all()) and bool((room[64 + at + rows * cols:] == 7.0).all())
                room.fill_(7.0)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_written_over_an_operand(dt):
    for cols in COLS[dt]:
        rows = 100
        z = gen.randn((rows, cols), 73, DEV, dt, std=3.0)
        mask = gen.randn((rows, cols), 74, DEV, dt)
        for over in ("z", "mask"):
            print(f"[case] masked softmax {dt} [{rows}, {cols}] written over its {over}", flush=True)
            d = {"z": z.clone(), "mask": mask.clone()}
            H.run_vm(desc(dt), d, {"p": d[over]})
            check(d[over], z, mask, dt, (cols, over))


@pytest.mark.parametrize("dt,shape", [("f32", (1, 3, 300, 20011)), ("f32", (1, 3, 1500, 5000)), ("bf16", (2, 2, 300, 30205)), ("bf16", (1, 2, 1601, 8200))])
def test_shared_by_the_second_dim(dt, shape):
    """Rows of an index taken together; beyond 24 MB of mask in blocks of 64 rows, the last of which is not full."""
    print(f"[case] masked softmax {dt} {list(shape)} under {list(shape[2:])}", flush=True)
    z = gen.randn(shape, 75, DEV, dt, std=3.0)
    mask = gen.randn(shape[2:], 76, DEV, dt)
    n = z.numel()
    room = torch.full((n + 128,), 7.0, dtype=z.dtype, device=DEV)
    out = room[64: 64 + n].view(shape)
    H.run_vm(desc(dt), {"z": z, "mask": mask}, {"p": out})
    for b in range(shape[0]):
        for h in range(shape[1]):
            check(out[b, h], z[b, h], mask, dt, (shape, b, h))
    assert bool((room[:64] == 7.0).all()) and bool((room[64 + n:] == 7.0).all())
