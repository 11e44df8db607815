"""Sums and differences with a product of two inputs that rides along in their record: every sign, tile registers enough and too
few (inputs loaded again), views, ragged rows, both types, against the oracle; and programs that must not lose a plan to it."""
from __future__ import annotations

from dataclasses import replace

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W
from workloads.programs import _p

from . import harness as H
from .test_written_inputs_cpu import make

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _ctx(k, nr):
    c = B.Context(torch.cuda.current_device())
    c.set_limits(k, nr)
    c.set_copies_in_flight(4096)            # (planned as part of a launch that fills the machine)
    return c


def forms(dt):
    ins = [("a", dt), ("b", dt), ("c", dt), ("d", dt)]
    ab, cd = ("p", "mul", ["a", "b"], {}), ("q", "mul", ["c", "d"], {})
    ex = ("p", "tanh", ["a"], {})
    return [_p("add", ins, [ab, cd, ("y", "add", ["p", "q"], {})], [("y", dt)]),
            _p("sub", ins, [ab, cd, ("y", "sub", ["p", "q"], {})], [("y", dt)]),
            _p("rsub", ins, [("q", "mul", ["c", "d"], {}), ex, ("s", "sub", ["q", "p"], {}), ("y", "add", ["s", "b"], {})], [("y", dt)]),
            _p("square", ins, [ab, ("q", "mul", ["c", "c"], {}), ("s", "add", ["p", "q"], {}), ("y", "mul", ["s", "d"], {})], [("y", dt)]),
            _p("kept", ins, [ab, cd, ("y", "add", ["p", "q"], {})], [("y", dt), ("q", dt)]),         # the product is an output too
            _p("norm", ins, [ab, cd, ("s", "add", ["p", "q"], {}), ("m", "rmax", ["s"], {}), ("y", "sub", ["s", "m"], {})], [("y", dt)])]


@pytest.mark.parametrize("limits", [(64, 6), (16, 4), (32, 2)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(33, 64), (7, 515), (3, 5000)])
def test_forms(shape, dt, limits):
    print(f"[case] products that ride along {dt} {shape} {limits}", flush=True)
    ctx = _ctx(*limits)
    d = {n: gen.randn(shape, 70 + i, DEV, dt) for i, n in enumerate("abcd")}
    d["d"] = gen.randn((shape[-1],), 75, DEV, dt)           # broadcast over the rows
    texts = []
    for desc in forms(dt):
        _, code, _ = H.check_program(desc, d, ctx=ctx)
        texts.append(code.disasm())
    assert any(" mac " in t for t in texts)


@pytest.mark.parametrize("limits", [(64, 6), (16, 4), (32, 2)])
def test_rope(limits):
    print(f"[case] RoPE {limits}", flush=True)
    d = gen.c5_inputs(37, 76, DEV)["c5_rope"]
    out = torch.empty((37, 32, 128), dtype=torch.bfloat16, device=DEV)
    _, code, _ = H.check_program(W.get_program("c5_rope"), d, outputs={"y1": out[..., :64], "y2": out[..., 64:]}, ctx=_ctx(*limits))
    assert " mac " in code.disasm() and code.info().variant_nr <= 4


def equal_bits(desc, d):
    """The program planned for a launch of its own and for one that fills the machine."""
    alone, _ = H.run_vm(desc, d, ctx=B.Context(torch.cuda.current_device()))
    full, code = H.run_vm(desc, d, ctx=_ctx(32, 6))
    for n, t in alone.items():
        a, b = (x.view(torch.int16 if x.dtype == torch.bfloat16 else torch.int32) for x in (t, full[n]))
        assert torch.equal(a, b), (desc.name, n)
    return code


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_the_size_of_the_launch_does_not_change_the_rounding(dt):
    print(f"[case] products that ride along, alone and in a full launch {dt}", flush=True)
    d = {n: gen.randn((33, 64), 70 + i, DEV, dt) for i, n in enumerate("abcd")}
    f32 = [replace(f, outputs=tuple((o, "f32") for o, _ in f.outputs)) for f in forms(dt) if f.name != "norm"]
    ab_cd = [("p", "mul", ["a", "b"], {}), ("q", "mul", ["c", "d"], {})]
    swapped = _p("swapped", f32[0].inputs, ab_cd + [("y", "add", ["q", "p"], {})], [("y", "f32")])
    between = _p("between", f32[0].inputs, ab_cd + [("t", "tanh", ["a"], {}), ("s", "add", ["p", "q"], {}), ("y", "add", ["s", "t"], {})], [("y", "f32")])
    texts = [equal_bits(f, d).disasm() for f in f32 + [swapped, between]]
    assert sum(" mac " in t for t in texts) >= 3
    # a difference of equal products is zero
    zero, code = H.run_vm(f32[1], {"a": d["a"], "b": d["b"], "c": d["a"], "d": d["b"]}, ctx=_ctx(32, 6))
    assert " mac " in code.disasm() and not zero["y"].any()


def test_random_programs_round_alike_in_every_launch():
    ran = 0
    for seed in range(120):
        desc = make(seed)
        if any(o.name in ("rmax", "sum") for o in desc.ops):        # (row plans may differ in the order of a sum)
            continue
        print(f"[case] random program {seed}, alone and in a full launch", flush=True)
        equal_bits(desc, {n: gen.randn((33, 512), 500 + 7 * seed + i, DEV, dt, std=0.5) for i, (n, dt) in enumerate(desc.inputs)})
        ran += 1
    assert ran > 30


def test_one_register_is_still_enough():
    """Two registers at once are more than this program needs without the record."""
    print("[case] a product and an exponential under one tile register", flush=True)
    desc = _p("one", [("c", "f32"), ("d", "f32"), ("x", "f32")], [("q", "mul", ["c", "d"], {}), ("e", "exp", ["x"], {}), ("y", "add", ["e", "q"], {})], [("y", "f32")])
    H.check_program(desc, {n: gen.randn((40, 300), 77 + i, DEV) for i, n in enumerate("cdx")}, ctx=_ctx(64, 1))
