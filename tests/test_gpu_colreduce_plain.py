"""Plain reductions along the penultimate axis (their own kernel): widths around a 16-byte piece and a column tile, few and
many units, fewer rows than lanes, strided operands, special values, both result types; against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads.programs import _p

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
SHAPES = [(1, 2, 3), (1, 2, 8), (1, 3, 9), (3, 5, 4), (2, 17, 33), (1, 1000, 65), (700, 7, 64), (5, 64, 2049), (1, 5003, 31), (2, 129, 515), (1, 70, 40000)]


def one(op, dt, out):
    return _p(f"plain_{op}", [("x", dt)], [("s", op, ["x"], {})], [("s", out)])


def check(op, dt, out, x):
    """Maxima and minima exactly (rounded to the result type).  Sums: a lane adds at most size / 4 rows one after the other (four waves at least share them), then
    come at most 6 steps across lanes and 16 waves: (size / 4 + 24) * 2^-24 of the sum of magnitudes, plus the result's rounding."""
    outs, _ = H.run_vm(one(op, dt, out), {"x": x})
    got, x64 = H.to_np64(outs["s"]), H.to_np64(x)
    if op != "csum":
        ref = getattr(np, "max" if op == "cmax" else "min")(x64, axis=-2, keepdims=True)
        np.testing.assert_array_equal(got, H.to_np64(torch.from_numpy(ref).to(outs["s"].dtype)))
        return
    with np.errstate(invalid="ignore"):
        ref, mag = x64.sum(-2, keepdims=True), np.abs(x64).sum(-2, keepdims=True)
    fin = np.isfinite(ref)
    np.testing.assert_array_equal(got[~fin], ref[~fin])
    tol = (x.shape[-2] / 4 + 24) * 2.0 ** -24 * mag + (2.0 ** -8 * np.abs(ref) if out == "bf16" else 0.0)
    assert np.all(np.abs(got - ref)[fin] <= tol[fin]), (op, dt, out, tuple(x.shape))


@pytest.mark.parametrize("dt,out", [("f32", "f32"), ("bf16", "f32"), ("bf16", "bf16"), ("f32", "bf16")])
@pytest.mark.parametrize("shape", SHAPES)
def test_shapes(shape, dt, out):
    print(f"[case] plain column reductions {dt} -> {out} {shape}", flush=True)
    x = gen.randn(shape, 51, DEV, dt)
    for op in ("csum", "cmax", "cmin"):
        check(op, dt, out, x)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_strided_operands_and_special_values(dt):
    print(f"[case] plain column reductions, views and special values {dt}", flush=True)
    base = gen.randn((4, 3, 90, 77), 52, DEV, dt)
    for v in (base[:, :, 5:80, 3:70], base.transpose(0, 1), base[::2], base[:, 1:, ::3, :21]):
        check("csum", dt, "f32", v)
    x = gen.randn((2, 300, 41), 53, DEV, dt)
    x[0, 7, 3] = float("nan")
    x[0, 299, 40] = float("inf")
    x[1, :, 11] = float("-inf")
    x[1, 150, 12] = float("-inf")
    for op in ("csum", "cmax", "cmin"):
        check(op, dt, "f32", x)


@pytest.mark.parametrize("shape", [(300, 20, 257), (300, 20, 256), (40, 300, 129), (1, 900, 33), (2, 64, 515)])
def test_written_over_the_first_row_of_the_input(shape):
    """Also where the row's last 16-byte piece slides back into the column tile before (257 fp32 columns in tiles of 256)."""
    for dt in ("f32", "bf16"):
        print(f"[case] column sum over row 0 of its input {dt} {shape}", flush=True)
        x = gen.randn(shape, 54, DEV, dt)
        ref, _ = H.run_vm(one("csum", dt, dt), {"x": x})
        mine = x.clone()
        H.run_vm(one("csum", dt, dt), {"x": mine}, outputs={"s": mine[:, :1, :]})
        assert torch.equal(mine[:, :1, :], ref["s"]) and torch.equal(mine[:, 1:, :], x[:, 1:, :])


def test_bytecode_without_outer_indices():
    """Valid bytecode over [0, 7, 64] that keeps the row length: nothing to do, and no launch of an empty grid."""
    print("[case] plain column reduction of no units", flush=True)
    x, s = gen.randn((3, 7, 64), 55, DEV), torch.full((3, 1, 64), -7.0, device=DEV)
    code = B.encode_for(H.gpu_ctx(), H.program(one("csum", "f32", "f32")), [x])
    w = np.frombuffer(code.raw, dtype=np.uint32).copy()
    seg = 8 + 3 * 2                     # behind the program header and two tensor entries
    assert w[seg + 9] == 21 and w[seg + 26] == 7
    w[seg + 2] = w[seg + 9] = 0         # tiles, rows
    empty = B.Bytecode(w.tobytes(), code.out_shapes)
    empty.validate()
    B.run_on(H.gpu_ctx(), empty, [x, s])
    torch.cuda.synchronize()
    assert bool((s == -7.0).all())
