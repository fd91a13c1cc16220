"""The order of a pass's work list (nearest tiles first in a batch of up to 65,536
atoms, by cost beyond) changes no output: systems evaluated alone, in a batch that
just fits the limit and in one just beyond it are equal bit for bit, and agree
with the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_common import build, compare_system, gpu_eval, params_pair

pytestmark = pytest.mark.gpu

LIMIT = 65536


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_list_order_changes_nothing(prec):
    first = [synth.make_system(200, 700, 11.8), synth.make_system(201, 321, 9.0)]
    filler = synth.make_system(202, 4001, 21.0)
    room = LIMIT - sum(s.n for s in first)
    fit = first + [filler] * (room // filler.n)
    last = synth.make_system(203, room % filler.n, 18.0)
    p = params_pair()[0]
    ref = None
    for systems in (first, fit + [last], fit + [last, synth.make_system(204, 1, 5.0)]):
        g, batch, plan, atoms = build(systems, prec)
        assert len(systems) == 2 or abs(plan.n_atoms - LIMIT) <= 1
        out = g.evaluate(plan, atoms, p)
        n = sum(s.n for s in first)
        got = {k: v[:2] if k.startswith("e_") else v[:n] for k, v in out.items()}
        if ref is None:
            ref = {k: v.clone() for k, v in got.items()}
            res = gpu_eval(plan, atoms, p)
            for b, s in enumerate(first):
                compare_system(res, b, batch.atom_offset, oracle.energy_forces(s, params_pair()[1]), prec)
        for k in ref:
            assert torch.equal(got[k], ref[k]), k
