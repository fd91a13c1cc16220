"""Small plans write their outputs from the pair passes: the energy pass forms the
Born radii of gb_evaluate, and the workgroup that counts a block's last item in
the chain pass writes the block's outputs.  Every subset of outputs, both entry
points, evaluation after evaluation on one workspace, under capture and after a
forked call: bitwise the plan with explicit work shapes, which runs a kernel of
its own for each of these; and the state that the Monte Carlo calls read."""
import itertools

import numpy as np
import pytest
import torch

import synth
from gpu_common import build, params_pair

pytestmark = pytest.mark.gpu

SIZES = [1, 64, 65, 200, 257]


def _plans(prec, sizes=SIZES):
    systems = [synth.make_system(180 + k, n, 18.0 * (max(n, 8) / 2500.0) ** (1 / 3))
               for k, n in enumerate(sizes)]
    g, batch, wide, atoms = build(systems, prec)
    _, _, walk, walk_atoms = build(systems, prec, j_blocks=1)
    return g, batch, wide, atoms, walk, walk_atoms


def _same(a, b):
    for k in a:
        assert (a[k] is None) == (b[k] is None)
        assert a[k] is None or torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_output_subsets(prec):
    g, _, wide, atoms, walk, walk_atoms = _plans(prec)
    p = params_pair()[0]
    for f, dq, dr in itertools.product([True, False], repeat=3):
        kw = dict(force=f, dEdq=dq, dEdrho=dr)
        _same(g.evaluate(wide, atoms, p, **kw), g.evaluate(walk, walk_atoms, p, **kw))
        assert torch.equal(g.radii(wide, atoms, p), g.radii(walk, walk_atoms, p))
        _same(g.energy_forces(wide, atoms, p, **kw), g.energy_forces(walk, walk_atoms, p, **kw))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_state_left_for_later_calls(prec):
    systems = [synth.make_system(190 + k, 237, 18.0 * (237 / 2500.0) ** (1 / 3), n_redox=1, n_prot=1)
               for k in range(3)]
    p = params_pair()[0]
    dE = []
    for tuning, fork in (({}, False), ({}, True), ({"j_blocks": 1}, False)):
        g, batch, plan, atoms = build(systems, prec, **tuning)
        sites = g.Sites.from_batch(plan, batch)
        cur = torch.as_tensor(batch.current_state, device=plan.device)
        side = torch.cuda.Stream()
        g.evaluate(plan, atoms, p, fork=side if fork else None)
        if fork:
            torch.cuda.current_stream().wait_stream(side)
        dE.append(g.mc_state_dE(plan, sites, atoms, cur, 7.0, np.full(3, -0.2), 300.0, p) +
                  tuple(g.energy_forces(plan, atoms, p).values()))
    for other in dE[1:]:
        for a, b in zip(dE[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_capture_and_replay(prec):
    g, _, wide, atoms, walk, walk_atoms = _plans(prec)
    p = params_pair()[0]
    g.evaluate(wide, atoms, p)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = g.evaluate(wide, atoms, p)
    for k in range(4):
        for a in (atoms, walk_atoms):
            a.x.mul_(1.01)
        graph.replay()
        torch.cuda.synchronize()
        _same(out, g.evaluate(walk, walk_atoms, p))
        # an eager call on the same workspace between replays
        _same(g.evaluate(wide, atoms, p), out)
