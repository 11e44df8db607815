"""Sums and differences with a product of two inputs that rides along in their record: every sign, tile registers enough and too
few (inputs loaded again), views, ragged rows, both types, against the oracle; and programs that must not lose a plan to it."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads import programs as W
from workloads.programs import _p

from . import harness as H

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


def test_one_register_is_still_enough():
    """Two registers at once are more than this program needs without the record."""
    print("[case] a product and an exponential under one tile register", flush=True)
    desc = _p("one", [("c", "f32"), ("d", "f32"), ("x", "f32")], [("q", "mul", ["c", "d"], {}), ("e", "exp", ["x"], {}), ("y", "add", ["e", "q"], {})], [("y", "f32")])
    H.check_program(desc, {n: gen.randn((40, 300), 77 + i, DEV) for i, n in enumerate("cdx")}, ctx=_ctx(64, 1))
