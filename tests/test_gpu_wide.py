"""The passes of small plans, which run one workgroup per work item, against the
same passes run one wavefront per item (a plan with explicit work shapes):
equal bit for bit in every output, whatever the launch.  Systems with one and
two rows of blocks, ragged blocks, lanes past the end, tiles with more marked
pairs than one round takes, separated tiles, several systems, salt, with and
without gradients; and the oracle on one of them."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_common import build, compare_system, gpu_eval, params_pair

pytestmark = pytest.mark.gpu


def _systems(sizes, squeeze=1.0):
    out = []
    for k, n in enumerate(sizes):
        s = synth.make_system(160 + k, n, 18.0 * (max(n, 8) / 2500.0) ** (1 / 3))
        for c in ("x", "y", "z"):
            setattr(s, c, synth.f32(getattr(s, c) * squeeze))
        out.append(s)
    return out


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes,squeeze,order", [
    ([1], 1.0, False), ([2, 63, 64, 65], 1.0, False), ([127, 128, 129, 191, 193], 1.0, False),
    ([256, 200], 0.55, False),          # 512 and more overlapping pairs per tile
    ([700], 1.0, True), ([1300], 1.0, True)])
@pytest.mark.parametrize("kappa", [0.0, 0.1])
def test_wide_equals_walk(prec, sizes, squeeze, order, kappa):
    systems = _systems(sizes, squeeze)
    p = dataclasses.replace(params_pair()[0], kappa=kappa)
    g, batch, wide, atoms = build(systems, prec)
    _, _, walk, walk_atoms = build(systems, prec, j_blocks=1)
    if order:
        o = g.block_order(batch.atom_offset, batch.x, batch.y, batch.z)
        wide.set_order(o)
        walk.set_order(o)
    a, b = g.evaluate(wide, atoms, p), g.evaluate(walk, walk_atoms, p)
    for k in a:
        assert torch.equal(a[k], b[k]), k
    for plan, at in ((wide, atoms), (walk, walk_atoms)):
        g.radii(plan, at, p)
    a, b = (g.energy_forces(q, at, p, force=False, dEdq=False, dEdrho=False)
            for q, at in ((wide, atoms), (walk, walk_atoms)))
    assert torch.equal(a["e_coul"], b["e_coul"]) and torch.equal(a["e_gb"], b["e_gb"])


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_wide_against_oracle(prec):
    systems = _systems([65, 300, 129])
    p_gpu, p_or = params_pair()
    g, batch, plan, atoms = build(systems, prec)
    res = gpu_eval(plan, atoms, p_gpu)
    for b, s in enumerate(systems):
        compare_system(res, b, batch.atom_offset, oracle.energy_forces(s, p_or), prec)


def test_wide_overflow_flag():
    # charges far outside the fixed-point range raise the flag there too
    systems = _systems([128])
    g, batch, plan, _ = build(systems, "fp32")
    atoms = g.Atoms(plan, batch.x, batch.y, batch.z, np.full(128, 1e9), batch.rho, batch.screen)
    g.evaluate(plan, atoms, params_pair()[0])
    assert g.check_overflow(plan)
    g.evaluate(plan, g.Atoms.from_batch(plan, batch), params_pair()[0])
    assert not g.check_overflow(plan)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n_systems", [896, 897, 1024, 1025])
def test_batches_of_single_blocks(prec, n_systems):
    # no tile off the diagonal: on both sides of the lines of such batches
    few = _systems([8, 3, 17, 64])
    systems = [few[k % 4] for k in range(n_systems)]
    g, batch, wide, atoms = build(systems, prec)
    _, _, walk, walk_atoms = build(systems, prec, j_blocks=1)
    a, b = g.evaluate(wide, atoms, params_pair()[0]), g.evaluate(walk, walk_atoms, params_pair()[0])
    for k in a:
        assert torch.equal(a[k], b[k]), k
