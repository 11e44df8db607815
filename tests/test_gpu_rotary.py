"""Rotations of pairs (RoPE) in the kernel of their own: the bits are the interpreter's, which runs the same bytecode as a part of a stack, in every
form the encoder gives them, over lane counts, shared and full tables, types, layouts and batched launches; and against float64."""
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


def rope(dt, tdt, swapped=False):
    """y1 = x1 c - x2 s, y2 = x2 c + x1 s; swapped: with the factors and summands the other way round."""
    ops = [("a", "mul", ["x1", "c"], {}), ("b", "mul", ["x2", "s"], {}), ("y1", "sub", ["a", "b"], {}),
           ("d", "mul", ["x2", "c"], {}), ("e", "mul", ["x1", "s"], {}), ("y2", "add", ["d", "e"], {})]
    if swapped:
        ops = [("a", "mul", ["c", "x1"], {}), ("b", "mul", ["s", "x2"], {}), ("d", "mul", ["c", "x2"], {}), ("e", "mul", ["s", "x1"], {}),
               ("y2", "add", ["e", "d"], {}), ("y1", "sub", ["a", "b"], {})]
    return W._p(f"rope_{dt}_{tdt}_{int(swapped)}", [("x1", dt), ("x2", dt), ("c", tdt), ("s", tdt)], ops, [("y1", dt), ("y2", dt)])


def tensors(T, heads, half, dt, tdt, shared):
    x = gen.randn((T, heads, 2 * half), 31, DEV, dt)
    t = [gen.randn((T, 1 if shared else heads, half), 32 + k, DEV, tdt) for k in range(2)]
    return {"x1": x[..., :half], "x2": x[..., half:], "c": t[0], "s": t[1]}


def check(got, d, dt):
    """Every product, and their sum or difference, rounds once in 32 bits: an error of at most 2^-24 (|p| + |q| + |p +- q|), so 2^-23 (|p| + |q|); a
    bf16 result (8 significant bits) rounds by 2^-8 of itself on top."""
    x1, x2, c, s = (d[n].double() for n in ("x1", "x2", "c", "s"))
    for y, p, q in ((got["y1"], x1 * c, -(x2 * s)), (got["y2"], x2 * c, x1 * s)):
        bound = 2.0 ** -23 * (p.abs() + q.abs())
        if dt == "bf16":
            bound = bound + 2.0 ** -8 * ((p + q).abs() + bound)
        worst = float(((y.double() - (p + q)).abs() / bound.clamp_min(1e-300)).max())
        assert worst <= 1.0


def bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("limits", [(64, 6), (16, 4), (32, 2), (8, 6)])
@pytest.mark.parametrize("dt,tdt", [("bf16", "f32"), ("bf16", "bf16"), ("f32", "f32")])
def test_alone_and_in_a_stack(dt, tdt, limits):
    ctx = B.Context(torch.cuda.current_device())
    ctx.set_limits(*limits)
    ctx.set_copies_in_flight(4096 if limits[1] < 6 else 1)      # (few registers: as a launch that fills the machine is encoded)
    stream = torch.cuda.current_stream().cuda_stream
    # (lanes on a row 1 to 64; heads that fill a wave's share of rows, and that do not; rows that end inside one)
    for T, heads, half, shared, swapped in ((37, 32, 64, True, False), (37, 32, 64, True, True), (300, 32, 64, True, False), (5, 3, 64, True, False), (7, 32, 64, False, False),
                                            (11, 256, 8, True, False), (9, 8, 256, True, False), (3, 5, 32, False, True), (1, 1, 8, True, False), (2, 16, 128, True, False),
                                            (900, 32, 64, True, False)):
        if limits[1] == 2 and (swapped or T * heads * half * 4096 <= 256 * 4 * 3 * 64 * 16):      # (two registers do not hold these forms)
            continue
        print(f"[case] rotation {dt} {tdt} {limits}: {T} x {heads} x 2 x {half}, tables {'shared' if shared else 'full'}", flush=True)
        desc = rope(dt, tdt, swapped)
        d = tensors(T, heads, half, dt, tdt, shared)
        room = [torch.full((T, heads, 2 * half + 8), 7.0, dtype=d["x1"].dtype, device=DEV) for _ in range(2)]
        outs = [{"y1": r[..., :half], "y2": r[..., half: 2 * half]} for r in room]
        H.run_vm(desc, d, outs[0], ctx=ctx)
        check(outs[0], d, dt)
        assert bool((room[0][..., 2 * half:] == 7.0).all())
        ins = [d[n] for n in ("x1", "x2", "c", "s")]
        code = B.encode_for(ctx, H.program(desc), ins, list(outs[1].values()))
        a = gen.randn((33,), 40, DEV)
        y = torch.empty_like(a)
        other = B.encode_for(ctx, H.program(W.single_op_program("abs", 1, "f32")), [a])
        ptrs = [t.data_ptr() for t in ins + list(outs[1].values()) + [a, y]]
        B.dvm_run(ctx, B.dvm_stack([code, other]), ptrs, stream)
        torch.cuda.synchronize()
        assert torch.equal(bits(room[0]), bits(room[1]))


def test_batched_and_written_inputs():
    T, n = 130, 3
    ctx = B.Context(torch.cuda.current_device())
    ctx.set_copies_in_flight(n)
    stream = torch.cuda.current_stream().cuda_stream
    sets = [tensors(T, 32, 64, "bf16", "f32", True) for _ in range(n)]
    for k, d in enumerate(sets):
        d["x1"].copy_(gen.randn((T, 32, 64), 50 + k, DEV, "bf16"))
    desc = rope("bf16", "f32")
    refs, outs = [], [torch.empty((T, 32, 128), dtype=torch.bfloat16, device=DEV) for _ in range(n)]
    for d in sets:
        y = torch.empty((T, 32, 128), dtype=torch.bfloat16, device=DEV)
        check(H.run_vm(desc, d, {"y1": y[..., :64], "y2": y[..., 64:]}, ctx=ctx)[0], d, "bf16")
        refs.append(y)
    ins = [[d[k] for k in ("x1", "x2", "c", "s")] + [y[..., :64], y[..., 64:]] for d, y in zip(sets, outs)]
    code = B.encode_for(ctx, H.program(desc), ins[0][:4], ins[0][4:])
    table = torch.empty(6 * n, dtype=torch.int64, device=DEV)
    print("[case] rotation in a batched launch", flush=True)
    B.dvm_run_batched(ctx, code, [[t.data_ptr() for t in s] for s in ins], table.data_ptr(), table.numel() * 8, stream)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(outs, refs))
    # Written over its inputs, in the form that allows it (all products first): the interpreter's, whose plan loads before it stores
    print("[case] rotation written over its inputs", flush=True)
    products = [("a", "mul", ["x1", "c"], {}), ("b", "mul", ["x2", "s"], {}), ("d", "mul", ["x2", "c"], {}), ("e", "mul", ["x1", "s"], {})]
    desc, d = W._p("rope_late", desc.inputs, products + [("y1", "sub", ["a", "b"], {}), ("y2", "add", ["d", "e"], {})], desc.outputs), sets[0]
    ins, whole = [d[k] for k in ("x1", "x2", "c", "s")], torch.empty_like(refs[0])
    views = [whole[..., :64], whole[..., 64:]]
    ctx.set_copies_in_flight(1)
    apart, over = B.encode_for(ctx, H.program(desc), ins, views), B.encode_for(ctx, H.program(desc), ins, ins[:2])
    assert [l.kind for l in L.launches(apart, [[t.data_ptr() for t in ins + views]])] == [L.ROTARY]
    assert [l.kind for l in L.launches(over, [[t.data_ptr() for t in ins + ins[:2]]])] == [L.INTERPRETER]
    B.run_on(ctx, apart, ins + views)
    B.run_on(ctx, over, ins + ins[:2])
    torch.cuda.synchronize()
    assert torch.equal(d["x1"], views[0]) and torch.equal(d["x2"], views[1])
