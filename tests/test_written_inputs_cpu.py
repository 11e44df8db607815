"""A call may write an output over an input of the same layout that no operator behind the one computing that output takes
(dvm_prog_output): in the encoded body every load of such an input precedes the store.  Random programs of several outputs,
small and large launches, few and many tile registers; read back from the disassembly."""
from __future__ import annotations

import re

import numpy as np
import pytest

from paper_2603_24239_amd import binding as B
from workloads.programs import _p

SHAPES = [(64, 1024), (16384, 1024), (512, 257), (300, 40000)]


def make(seed):
    rng = np.random.default_rng(seed)
    inputs = [(f"i{k}", "f32" if rng.integers(0, 2) else "bf16") for k in range(int(rng.integers(2, 7)))]
    vals, ops = [n for n, _ in inputs], []

    def pick():
        return str(rng.choice(vals[-7:] if rng.integers(0, 2) else vals))
    for k in range(int(rng.integers(3, 14))):
        r, o = int(rng.integers(0, 10)), f"v{k}"
        if r < 7:
            ops.append((o, "mul" if r < 4 else str(rng.choice(["add", "sub"])), [pick(), pick()], {}))
        elif r < 8:
            ops.append((o, "exp", [pick()], {}))
        elif r < 9:
            ops.append((o, str(rng.choice(["rmax", "sum"])), [pick()], {}))
        else:
            ops.append((o, "square", [pick()], {}))
        vals.append(o)
    names = [o[0] for o in ops]
    outs = dict.fromkeys([names[-1]] + [str(x) for x in rng.choice(names, min(3, len(names)), replace=False)])
    return _p(f"multi_{seed}", inputs, ops, [(o, "f32") for o in outs])


def late_loads(desc, code):
    """(output, input) pairs whose load comes behind the store although no later operator takes the input."""
    n_in = len(desc.inputs)
    at = {o.out: i for i, o in enumerate(desc.ops)}
    last = [max([i for i, o in enumerate(desc.ops) if n in o.args], default=-1) for n, _ in desc.inputs]
    stored, late = [], []
    for line in code.disasm().splitlines():
        m = re.match(r"\s+\d{4} (\S*load\S*|\S*store\S*)\s.*?\bt(\d+)\b", line)
        if not m:
            continue
        t = int(m.group(2))
        if "store" in m.group(1):
            stored.append(t - n_in)
        else:
            late += [(o, t) for o in stored if last[t] <= at[desc.outputs[o][0]]]
    return late


def contexts():
    for limits, copies in (((32, 6), 1), ((16, 4), 1), ((64, 6), 32)):
        c = B.Context(-1)
        c.set_limits(*limits)
        c.set_copies_in_flight(copies)
        yield c


def test_random_programs_load_an_input_before_the_stores_behind_its_last_use():
    n = 0
    ctxs = list(contexts())
    for seed in range(400):
        desc = make(seed)
        prog = B.Program(desc)
        for c in ctxs:
            for shape in SHAPES:
                try:
                    code = B.dvm_encode(c, prog, [B.make_shape(shape)] * len(desc.inputs))
                    code.validate()
                except B.DvmError:
                    continue
                n += 1
                assert not late_loads(desc, code), (seed, shape)
    assert n > 4000


FORMS = {
    # a product of two inputs taken by a later difference (I_MAC in large launches), an output stored in between
    "product": ([("p", "mul", ["a", "b"], {}), ("t", "exp", ["b"], {}), ("q", "mul", ["x", "y"], {}), ("r", "sub", ["q", "p"], {})], ["t", "r"]),
    # exp(a - b) and sum(square(a)), fused into one record each, likewise
    "expsub": ([("d", "sub", ["a", "b"], {}), ("t", "mul", ["x", "y"], {}), ("r", "exp", ["d"], {})], ["t", "r"]),
    "sumsq": ([("d", "square", ["a"], {}), ("t", "mul", ["x", "y"], {}), ("s", "sum", ["d"], {}), ("r", "add", ["t", "s"], {}), ("z", "add", ["r", "b"], {})], ["t", "z"]),
}


@pytest.mark.parametrize("form", FORMS)
def test_fusions_do_not_move_a_load_behind_a_store(form):
    ops, outs = FORMS[form]
    desc = _p(form, [(n, "f32") for n in "abxy"], ops, [(o, "f32") for o in outs])
    for c in contexts():
        for shape in SHAPES[:3]:
            code = B.dvm_encode(c, B.Program(desc), [B.make_shape(shape)] * 4)
            assert not late_loads(desc, code), (form, shape)
    # without the output in between they are fused as ever
    alone = B.dvm_encode(next(contexts()), B.Program(_p(form, desc.inputs, ops, [(outs[1], "f32")])), [B.make_shape((16384, 1024))] * 4)
    assert {"product": " mac ", "expsub": "expsub", "sumsq": "red.sumsq"}[form] in alone.disasm()


def test_a_program_that_only_fits_the_registers_fused_is_still_accepted():
    c = B.Context(-1)
    c.set_limits(64, 1)
    ops, outs = FORMS["expsub"]
    desc = _p("tight", [(n, "f32") for n in "abxy"], ops, [(o, "f32") for o in outs])
    code = B.dvm_encode(c, B.Program(desc), [B.make_shape((64, 1024))] * 4)
    code.validate()
    assert "expsub" in code.disasm()
