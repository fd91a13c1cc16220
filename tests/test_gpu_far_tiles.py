"""GPU parity on tiles at the edge of the shortest fits: two compact blocks of
64 atoms whose boxes just clear the distance at which (S/r)^2 stays within
their domain on every pair, and just miss it (the fits of the nearer separated
tiles); one and two rows of blocks, in both plans, walked by one wavefront and
by one workgroup per item, which agree bit for bit."""
import os
import re

import numpy as np
import pytest
import torch

import synth
from gpu_common import build, compare_system, gpu_eval, oracle_eval, params_pair

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1803_09652_amd", "csrc")
YVFAR = float(re.search(r"#define GBMC_HCT_YVFAR ([\d.]+)f",
                        open(os.path.join(CSRC, "hct_vfar.inc")).read()).group(1))
OFFSET = 0.09          # IGB5 offset (A)


def _clusters(blocks, stretch):
    """`blocks` 64-atom clusters along x, neighbours `stretch` times the rule's
    distance apart; and the largest y over pairs of neighbours."""
    parts = [synth.make_system(31 + k, 64, 3.5) for k in range(blocks)]
    xyz = [p.coords().astype(np.float64) for p in parts]
    S = [p.screen * (p.rho - OFFSET) for p in parts]
    gap = max(s.max() for s in S) / np.sqrt(0.999 * YVFAR) * stretch
    for a, b in zip(xyz, xyz[1:]):
        b[:, 0] += a[:, 0].max() - b[:, 0].min() + gap
    ymax = 0.0
    for k in range(blocks - 1):
        r2 = ((xyz[k][:, None] - xyz[k + 1][None]) ** 2).sum(-1)
        ymax = max(ymax, (S[k][:, None] ** 2 / r2).max(), (S[k + 1][None] ** 2 / r2).max())
    x = synth.f32(np.concatenate(xyz))
    cat = lambda c: np.concatenate([getattr(p, c) for p in parts])
    return synth.System(x[:, 0].copy(), x[:, 1].copy(), x[:, 2].copy(), cat("q"), cat("rho"),
                        cat("screen")), ymax


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("blocks", [2, 3, 5])
@pytest.mark.parametrize("stretch", [1.002, 0.998])
def test_edge_of_the_shortest_fits(prec, blocks, stretch):
    s, ymax = _clusters(blocks, stretch)
    assert 0.5 * YVFAR < ymax <= YVFAR                 # the upper part of the fits' range
    p_gpu, p_or = params_pair()
    ref = oracle_eval(s, p_or)
    out = []
    for tuning in ({}, {"j_blocks": 1}, {"j_blocks": 8}):
        g, batch, plan, atoms = build([s], prec, **tuning)
        out.append(g.evaluate(plan, atoms, p_gpu))
        compare_system(gpu_eval(plan, atoms, p_gpu), 0, batch.atom_offset, ref, prec)
    for k in out[0]:
        assert torch.equal(out[0][k], out[1][k]) and torch.equal(out[0][k], out[2][k]), k
