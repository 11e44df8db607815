"""Softmax along the row in the kernel of its own: rows at the edges of its lane counts and slots of chunks, at every place in a 128-byte line,
with and without a second tensor, against float64; equal bits wherever a row stands, in place, in a stack and in a batched launch."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
INF = float("inf")
MIN_BYTES = 16 << 20        # below, a program that is nothing else runs in the kernel with the interpreter's bits, a part of a stack in the interpreter
TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
# lanes on a row change behind 258, 578, 1218 (bf16; in fp32 back and forth, 128 behind 2018) and on up to 512; a workgroup keeps a row behind 16353 (24513),
# of 1024 lanes behind 49121 (65473); its slots leave the registers behind 32737, change their kernel behind 114657, and the kernel ends at 135137 (163777)
# columns that start anywhere in a line
EDGES = {"f32": [4, 5, 31, 33, 65, 97, 98, 225, 226, 481, 482, 1000, 1411, 2017, 2018, 2048, 4096, 8161, 8162, 8192, 16353, 16354, 32737, 32738, 49121, 49122, 60011, 114657, 114658,
                 131041, 131042, 131072, 135137, 135138],
         "bf16": [8, 9, 63, 65, 193, 194, 257, 449, 450, 751, 961, 962, 1985, 1986, 4096, 16321, 16322, 24513, 24514, 65473, 65474, 131071, 163777, 163778]}


def rows_for(cols, dt):
    es = 4 if dt == "f32" else 2
    return max(14, -(-MIN_BYTES // (2 * es * cols)) + 3)


def desc(dt, mask=False):
    if mask:
        return W._p(f"masked_softmax_{dt}", [("z", dt), ("mask", dt)], [("s", "add", ["z", "mask"], {}), ("p", "softmax", ["s"], {})], [("p", dt)])
    return W.get_program(f"softmax_{dt}")


def check(got, z, dt, what):
    """The exponential's argument carries a rounding of (z - max) * 2^-24, up to 1e-5 at the differences that matter; bf16 rounds once more."""
    ref = torch.softmax(z.double(), dim=-1)
    rel = 2e-5 if dt == "f32" else 2.0 ** -8 + 2e-5
    assert torch.equal(torch.isnan(got), torch.isnan(ref)), what
    err = (got.double() - ref).abs()
    tiny = 1e-37
    ok = torch.isnan(ref) | (err <= rel * ref + tiny)
    assert bool(ok.all()), (what, float((err / (ref + 1e-30)).nan_to_num().max()))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_edges(dt):
    for cols in EDGES[dt]:
        n = rows_for(cols, dt)
        print(f"[case] softmax {dt} [{n}, {cols}]", flush=True)
        z = gen.randn((13, cols), 11, DEV, dt, std=3.0)
        z[1] = -INF
        z[2, : cols // 2] = -INF
        z[3, cols - 1] = INF
        z[4, 0] = float("nan")
        z[5, cols - 1] = float("nan")
        z[6] = torch.linspace(-60.0, 60.0, cols, device=DEV).to(z.dtype)
        x = z.repeat(-(-n // 13), 1)[:n].contiguous()
        got, _ = H.run_vm(desc(dt), {"z": x})
        y = got["p"]
        check(y[:13], z, dt, cols)
        bits = y.nan_to_num(-1.0).view(torch.int32 if dt == "f32" else torch.int16)
        assert torch.equal(bits, bits[:13].repeat(-(-n // 13), 1)[:n]), f"equal rows, different bits: {cols}"


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_places_in_a_line_and_in_place(dt):
    es = 4 if dt == "f32" else 2
    for cols in (67, 751, 5000, 40003):
        n = rows_for(cols, dt)
        z = gen.randn((n, cols), 12, DEV, dt, std=3.0)
        ref = H.run_vm(desc(dt), {"z": z})[0]["p"]
        for at_in, at_out in ((0, 1), (3, 0), (128 // es - 1, 5), (7, 128 // es - 1)):
            print(f"[case] softmax {dt} [{n}, {cols}], input and output {at_in} and {at_out} elements into a line", flush=True)
            zi = torch.empty(n * cols + 64, dtype=z.dtype, device=DEV)[at_in: at_in + n * cols].view(n, cols)
            zi.copy_(z)
            room = torch.full((n * cols + 256,), 7.0, dtype=z.dtype, device=DEV)
            out = room[64 + at_out: 64 + at_out + n * cols].view(n, cols)
            H.run_vm(desc(dt), {"z": zi}, {"p": out})
            assert torch.equal(out, ref)
            assert bool((room[: 64 + at_out] == 7.0).all()) and bool((room[64 + at_out + n * cols:] == 7.0).all())
        print(f"[case] softmax {dt} [{n}, {cols}] in place", flush=True)
        zi = z.clone()
        H.run_vm(desc(dt), {"z": zi}, {"p": zi})
        assert torch.equal(zi, ref)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_second_tensor_and_strides(dt):
    for b, h, s in ((2, 3, 1411), (1, 5, 700), (3, 2, 2600)):
        z = gen.randn((b, h, s, s), 13, DEV, dt, std=3.0)
        causal = torch.zeros((s, s), device=DEV).masked_fill_(torch.ones((s, s), dtype=torch.bool, device=DEV).triu(1), -INF).to(z.dtype)
        bias = gen.randn((b, 1, s, s), 14, DEV, dt)
        for what, m in (("causal", causal), ("bias", bias), ("full", gen.randn((b, h, s, s), 15, DEV, dt)), ("row", bias[0, 0, 0])):
            print(f"[case] masked softmax {dt} {tuple(z.shape)}, {what} {tuple(m.shape)}", flush=True)
            got = H.run_vm(desc(dt, True), {"z": z, "mask": m})[0]["p"]
            check(got, z.float() + m.float(), dt, what)
        print(f"[case] strided softmax {dt}", flush=True)
        v = z.transpose(0, 2)[:, :, :, : s - 3]
        out = torch.full((s, h, b, s + 5), 7.0, dtype=z.dtype, device=DEV)
        H.run_vm(desc(dt), {"z": v}, {"p": out[..., 2: s - 1]})
        check(out[..., 2: s - 1], v, dt, "strided")
        assert bool((out[..., :2] == 7.0).all()) and bool((out[..., s - 1:] == 7.0).all())


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_stack_and_batch(dt):
    ctx = B.Context(torch.cuda.current_device())
    stream = torch.cuda.current_stream().cuda_stream
    for cols in (300, 1411, 20011):
        n = rows_for(cols, dt)
        print(f"[case] softmax {dt} [{n}, {cols}]: 3 sets, and 3 parts among others", flush=True)
        xs = [gen.randn((n, cols), 16 + i, DEV, dt, std=3.0) for i in range(3)]
        code = B.encode_for(ctx, H.program(desc(dt)), [xs[0]])
        refs = [torch.empty_like(x) for x in xs]
        for x, y in zip(xs, refs):
            B.run_on(ctx, code, [x, y])
        outs = [torch.full_like(x, -7.0) for x in xs]
        table = torch.empty(6, dtype=torch.int64, device=DEV)
        B.dvm_run_batched(ctx, code, [[x.data_ptr(), y.data_ptr()] for x, y in zip(xs, outs)], table.data_ptr(), 48, stream)
        assert all(torch.equal(a, b) for a, b in zip(outs, refs))
        a, c = gen.randn((999, 64), 20, DEV, dt), gen.randn((999, 64), 21, DEV, dt)
        add = W.single_op_program("add", 2, dt)
        add_code = B.encode_for(ctx, H.program(add), [a, c])
        sums = [torch.empty_like(a) for _ in range(2)]
        outs = [torch.full_like(x, -7.0) for x in xs]
        parts, ptrs = [], []
        for k in range(3):
            parts.append(code)
            ptrs += [xs[k].data_ptr(), outs[k].data_ptr()]
            if k < 2:
                parts.append(add_code)
                ptrs += [a.data_ptr(), c.data_ptr(), sums[k].data_ptr()]
        B.dvm_run(ctx, B.dvm_stack(parts), ptrs, stream)
        torch.cuda.synchronize()
        want = (a.float() + c.float()).to(a.dtype)
        assert all(torch.equal(p, q) for p, q in zip(outs, refs)) and all(torch.equal(p, want) for p in sums)


@pytest.mark.parametrize("limits", [(64, 1), (64, 6), (32, 2), (8, 6)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_small_programs_have_the_interpreters_bits(dt, limits):
    """Alone and batched they run in a kernel that adds in the interpreter's order; in a stack in the interpreter."""
    ctx = B.Context(torch.cuda.current_device())
    ctx.set_limits(*limits)
    stream = torch.cuda.current_stream().cuda_stream
    a = gen.randn((33,), 40, DEV)
    other = B.encode_for(ctx, H.program(W.single_op_program("abs", 1, "f32")), [a])
    for rows, cols in ((1, 3), (777, 1), (777, 3), (500, 7), (63, 8), (64, 9), (65, 26), (1000, 32), (300, 65), (257, 100), (129, 250), (130, 257), (40, 512), (33, 1000), (5, 2049), (3, 4096)):
        for masked in (False, True):
            if masked and limits[1] < 2:
                continue
            print(f"[case] softmax {dt} [{rows}, {cols}] {limits}{', masked' if masked else ''}", flush=True)
            z = gen.randn((3, rows, cols), 41, DEV, dt, std=3.0)
            z[:, 0, cols // 2] = -INF
            ins = [z] + ([gen.randn((rows, cols), 42, DEV, dt)] if masked else [])
            names = [n for n, _ in desc(dt, masked).inputs]
            alone = H.run_vm(desc(dt, masked), dict(zip(names, ins)), ctx=ctx)[0]["p"]
            check(alone, z.float() + ins[1].float() if masked else z, dt, (rows, cols))
            code = B.encode_for(ctx, H.program(desc(dt, masked)), ins)
            y, o = torch.empty_like(z), torch.empty_like(a)
            B.dvm_run(ctx, B.dvm_stack([code, other]), [t.data_ptr() for t in ins + [y, a, o]], stream)
            torch.cuda.synchronize()
            bits = [t.view(torch.int32 if dt == "f32" else torch.int16) for t in (alone, y)]
            assert torch.equal(*bits), (rows, cols, masked)
