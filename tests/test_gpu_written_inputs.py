"""Calls that write an output over an input no later operator takes, above the size at which products ride along with a sum
(I_MAC), give the bits of the same program writing elsewhere."""
from __future__ import annotations

import pytest
import torch

from paper_2603_24239_amd import binding as B
from workloads import gen
from workloads.programs import _p

from . import harness as H
from .test_written_inputs_cpu import FORMS

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("rows,cols", [(64, 1024), (4096, 1024), (4099, 1021)])
@pytest.mark.parametrize("form", FORMS)
def test_output_over_an_input(form, rows, cols):
    ops, outs = FORMS[form]
    desc = _p(form, [(n, "f32") for n in "abxy"], ops, [(o, "f32") for o in outs])
    ctx = B.Context(torch.cuda.current_device())
    ins = {n: gen.randn((rows, cols), 80 + i, DEV) for i, n in enumerate("abxy")}
    ref, _ = H.run_vm(desc, ins, ctx=ctx)
    first = next(i for i, o in enumerate(ops) if o[0] == outs[0])
    for name in "abxy":
        if any(name in o[2] for o in ops[first + 1:]):
            continue
        print(f"[case] {form} [{rows}, {cols}]: {outs[0]} over {name}", flush=True)
        mine = {n: t.clone() for n, t in ins.items()}
        got, _ = H.run_vm(desc, mine, outputs={outs[0]: mine[name], outs[1]: torch.empty_like(ref[outs[1]])}, ctx=ctx)
        for o in outs:
            assert torch.equal(got[o], ref[o]), (form, name, o)
