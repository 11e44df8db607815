"""Which kernel a run takes, and its launch: host rules, evaluated without a device over addresses that need not exist."""
from __future__ import annotations

import pytest

from paper_2603_24239_amd import binding as B
from workloads import programs as W

from . import launch_plan as L

ES = {"f32": 4, "bf16": 2}
FAR = 1 << 40       # between tensors


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(-1)
    c.set_planner(256)
    return c


def softmax(dt, masked=False):
    if masked:
        return B.Program(W._p(f"masked_{dt}", [("z", dt), ("m", dt)], [("s", "add", ["z", "m"], {}), ("p", "softmax", ["s"], {})], [("p", dt)]))
    return B.Program(W.get_program(f"softmax_{dt}"))


def encode(ctx, dt, shape, masked=False):
    return B.dvm_encode(ctx, softmax(dt, masked), [B.make_shape(shape, align_bytes=4)] * (1 + masked), [B.make_shape(shape, align_bytes=4)])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("cols", [25089, 30205, 65474, 131000])
def test_long_rows_written_over_an_operand(ctx, dt, cols):
    """Written over the first operand a row is read before it is stored.  The second one of a long bf16 row is read again beside the stores: such a call
    stays with the interpreter."""
    code = encode(ctx, dt, (100, cols), masked=True)
    z, m, y = FAR, 2 * FAR, 3 * FAR
    assert [l.kind for l in L.launches(code, [[z, m, y]])] == [L.SOFTMAX_LONG]
    assert [l.kind for l in L.launches(code, [[z, m, z]])] == [L.SOFTMAX_LONG]
    kept = L.INTERPRETER if dt == "bf16" else L.SOFTMAX_LONG
    assert [l.kind for l in L.launches(code, [[z, m, m]])] == [kept]
    assert [l.kind for l in L.launches(code, [[z, m, y], [z + 4096, m, m]])] == [kept]       # (in one set of a batch)
    plain = encode(ctx, dt, (100, cols))
    assert [l.kind for l in L.launches(plain, [[z, z]])] == [L.SOFTMAX_LONG]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_shorter_rows_written_over_either_operand(ctx, dt):
    code = encode(ctx, dt, (6000, 2600), masked=True)
    for y in (FAR, 2 * FAR, 3 * FAR):
        assert [l.kind for l in L.launches(code, [[FAR, 2 * FAR, y]])] == [L.SOFTMAX]
    for y in (FAR + 2600 * ES[dt], 2 * FAR + ES[dt]):           # (any other overlap)
        assert [l.kind for l in L.launches(code, [[FAR, 2 * FAR, y]])] == [L.INTERPRETER]


@pytest.mark.parametrize("dt,rows,cols,kind", [("f32", 1 << 29, 32, L.SOFTMAX), ("bf16", 1 << 29, 64, L.SOFTMAX), ("bf16", (1 << 29) - 31, 100, L.SOFTMAX),
                                               ("f32", (1 << 31) - 1, 3, L.SOFTMAX_EXACT), ("f32", 1 << 20, 1 << 13, L.SOFTMAX), ("f32", 1 << 13, 1 << 17, L.SOFTMAX_LONG)])
def test_a_launch_has_fewer_threads_than_it_may(ctx, dt, rows, cols, kind):
    """HIP takes fewer than 2^32 threads; the kernels stride over the tiles that are left."""
    (l,) = L.launches(encode(ctx, dt, (rows, cols)), [[FAR, 2 * FAR]])
    assert l.kind == kind and 0 < l.grid * l.block < 1 << 32


@pytest.mark.parametrize("tokens,kind", [(1 << 20, L.ROTARY), (1 << 25, L.INTERPRETER)])
def test_a_rotation_beyond_one_launch(ctx, tokens, kind):
    """Three heads of 2 * 512 columns under shared tables: a wave takes one row."""
    prog = B.Program(W.get_program("c5_rope"))
    x = B.make_shape((tokens, 3, 512), (3072, 1024, 1), 16)
    t = B.make_shape((tokens, 1, 512), (512, 512, 1), 16)
    code = B.dvm_encode(ctx, prog, [x, x, t, t], [x, x])
    q, c, s, y = FAR, 3 * FAR, 5 * FAR, 7 * FAR
    (l,) = L.launches(code, [[q, q + 1024, c, s, y, y + 1024]])
    assert l.kind == kind and l.grid * l.block < 1 << 32


# widths of whole lines whose lanes or kernel a row that starts inside a line would change
WHOLE_LINES = {"f32": [192, 448, 2048, 8160, 16384, 32768, 131072], "bf16": [448, 960, 1984, 16384, 24576, 65536, 163840]}


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_lanes_do_not_depend_on_addresses(ctx, dt):
    """The sums of a row, and so its bits, follow from its lanes; the kernel must be the same too, apart from its slots of chunks."""
    for cols in WHOLE_LINES[dt]:
        rows = -(-(20 << 20) // (2 * ES[dt] * cols))
        code = encode(ctx, dt, (rows, cols))
        (on,) = L.launches(code, [[FAR, 2 * FAR]])
        assert on.kind in (L.SOFTMAX, L.SOFTMAX_LONG)
        for at in (ES[dt] if dt == "f32" else 4, 16, 124):
            for sets in ([[FAR, 2 * FAR + at]], [[FAR + 64, 2 * FAR], [FAR, 2 * FAR + at], [FAR, 3 * FAR]]):
                (off,) = L.launches(code, sets)
                assert (off.kind, off.lanes, off.block) == (on.kind, on.lanes, on.block), (cols, at)
                assert on.slots <= off.slots <= on.slots + 1


def stacked(ctx, parts):
    codes = [encode(ctx, dt, shape, masked) for dt, shape, masked in parts]
    ptrs, at = [], FAR
    for _, _, masked in parts:
        for _ in range(2 + masked):
            ptrs.append(at)
            at += FAR
    return [(l.kind, l.n_segments, l.mixed) for l in L.launches(B.dvm_stack(codes), [ptrs])]


def test_softmaxes_of_a_stack_share_launches(ctx):
    """Groups of alike ones; groups too small to fill the chip together where type, second tensor and kernel are the same, wherever they stand."""
    a, b = ("f32", (16, 100003), False), ("f32", (17, 100011), False)
    assert stacked(ctx, [a, b, a, b]) == [(L.SOFTMAX_LONG, 4, 1)]
    assert stacked(ctx, [a, a, a]) == [(L.SOFTMAX_LONG, 3, 0)]
    short = ("bf16", (6000, 751), False), ("bf16", (14900, 300), False), ("bf16", (1500, 3000), False)
    add = ("bf16", (9, 64), False)                              # (small: with the interpreter, first)
    assert stacked(ctx, [short[0], add, short[1], a, short[2]]) == [(L.INTERPRETER, 1, 0), (L.SOFTMAX, 3, 1), (L.SOFTMAX_LONG, 1, 0)]
    large = ("bf16", (60000, 751), False)                       # (fills the chip)
    assert stacked(ctx, [short[0], large, short[1]]) == [(L.SOFTMAX, 2, 1), (L.SOFTMAX, 1, 0)]
    assert stacked(ctx, [short[0], short[1], short[0], short[1], short[0]]) == [(L.SOFTMAX, 3, 0), (L.SOFTMAX, 2, 0)]
    assert stacked(ctx, [a, ("bf16", (64, 40003), False), ("f32", (16, 100003), True), ("f32", (64, 17000), False)]) == [(L.SOFTMAX_LONG, 1, 0)] * 4


def test_the_fuser_counts_what_it_launches():
    """A softmax that runs apart among the pieces is a launch, though the bytecode does not ask for one (dvm_code_info.n_launches)."""
    ctx = B.Context(-1)
    ctx.set_limits(16, 2)           # (one interpreter variant for both pieces)
    for rows, launches in ((6000, 2), (600, 1)):
        f = B.Fuser(ctx)
        f.set_workspace(5 * FAR, 256)
        p = f.op("softmax", [f.tensor(FAR, "bf16", B.make_shape((rows, 751)))], "bf16", 2 * FAR)
        q = f.op("exp", [f.tensor(3 * FAR, "bf16", B.make_shape((rows, 753)))], "bf16", 4 * FAR)
        f.flush()
        assert f.last_code().info().n_segments == 2 and f.last_code().info().n_launches == 1 and p != q
        assert f.stats()["launches"] == launches, rows


@pytest.mark.parametrize("name,cols,n,reads", [("c2_rmsnorm", 4096, 2, 1), ("c4_chain", 8192, 6, 3), ("add_f16like", 4096, 2, 2), ("add_sqrt", 4096, 2, 2)])
def test_streaming_hint(ctx, name, cols, n, reads):
    """By the bytes that a launch reads: 96 MB, in bf16 32 of several tensors."""
    desc = W.get_program(name)
    es = ES[desc.inputs[0][1]]
    bound = (32 if reads > 1 and es == 2 else 96) << 20
    for rows, hint in ((bound // (reads * es * cols) - 3, 0), (bound // (reads * es * cols) + 1, 1)):
        shapes = [B.make_shape((cols,) if n_ in ("w", "gamma", "beta", "bias") else (rows, cols)) for n_, _ in desc.inputs]
        assert len(shapes) == n
        code = B.dvm_encode(ctx, B.Program(desc), shapes)
        (l,) = L.launches(code, [[FAR * (k + 1) for k in range(n + 1)]])
        assert l.kind == L.INTERPRETER and l.stream == hint, (rows, l.stream)
