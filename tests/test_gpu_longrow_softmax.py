"""Softmax over rows longer than a tile: the maximum and the sum of exponentials come from one pass.  Special values, maxima that
grow from tile to tile, the sum as an output, and forms that must keep their separate passes; against the oracle."""
from __future__ import annotations

import pytest
import torch

from workloads import gen
from workloads.programs import _p, single_op_program

from . import harness as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
INF = float("inf")


def rows(cols, dt):
    z = gen.randn((9, cols), 61, DEV, dt, std=3.0)
    z[1, :] = -INF
    z[2, : cols // 2] = -INF                        # whole tiles of -inf first
    z[3, cols // 2:] = -INF                         # ... and last
    z[4, 5] = INF
    z[5, cols - 1] = float("nan")
    z[6] = torch.linspace(-60.0, 60.0, cols, device=DEV).to(z.dtype)         # the maximum grows tile after tile
    z[7] = torch.linspace(60.0, -60.0, cols, device=DEV).to(z.dtype)
    return z


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("cols", [16387, 50001, 65536])
def test_special_rows(cols, dt):
    print(f"[case] long-row softmax {dt} [9, {cols}]", flush=True)
    _, code, _ = H.check_program(single_op_program("softmax", 1, dt), {"a0": rows(cols, dt)})
    assert "in one pass with the sum below" in code.disasm()


def test_the_sum_as_an_output_and_a_mask():
    print("[case] long-row softmax with its sum as an output", flush=True)
    desc = _p("lse", [("z", "f32"), ("mask", "f32")],
              [("s", "add", ["z", "mask"], {}), ("m", "rmax", ["s"], {}), ("d", "sub", ["s", "m"], {}), ("e", "exp", ["d"], {}), ("l", "sum", ["e"], {}),
               ("p", "div", ["e", "l"], {})], [("p", "f32"), ("l", "f32")])
    z = gen.randn((5, 33333), 62, DEV)
    mask = torch.zeros(33333, device=DEV)
    mask[20000:] = -INF
    _, code, _ = H.check_program(desc, {"z": z, "mask": mask})
    assert "in one pass with the sum below" in code.disasm()


def test_forms_that_take_separate_passes():
    print("[case] long rows: a minimum, and the exponential of another tensor", flush=True)
    softmin = _p("softmin", [("z", "f32")], [("m", "rmin", ["z"], {}), ("d", "sub", ["m", "z"], {}), ("e", "exp", ["d"], {}), ("l", "sum", ["e"], {}),
                                             ("p", "div", ["e", "l"], {})], [("p", "f32")])
    other = _p("other", [("z", "f32"), ("y", "f32")], [("m", "rmax", ["z"], {}), ("d", "sub", ["y", "m"], {}), ("e", "exp", ["d"], {}), ("l", "sum", ["e"], {}),
                                                       ("p", "div", ["e", "l"], {})], [("p", "f32")])
    z, y = gen.randn((4, 20001), 63, DEV), gen.randn((4, 20001), 64, DEV)
    for desc, ins in ((softmin, {"z": z}), (other, {"z": z, "y": y})):
        _, code, _ = H.check_program(desc, ins)
        assert "in one pass with the sum below" not in code.disasm()
