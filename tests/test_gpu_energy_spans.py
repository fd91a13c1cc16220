"""The energies of systems whose shares are summed in one or several spans of
4,096 atoms: whole and ragged spans, an empty system, and the same values from
the call that writes them after the energy pass and the one that writes them
after the chain pass, on repeated calls in one workspace (integer sums: equal
bit for bit), against the per-atom identity E_C + E_GB = 1/2 sum q dE/dq."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import build, params_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-6), ("fp64", 1e-10)])
def test_energy_sums_over_spans(prec, tol):
    sizes = [4095, 1, 4096, 4097, 8192, 8193]
    systems = [synth.make_system(150 + k, n, 18.0 * (max(n, 8) / 2500.0) ** (1 / 3)) for k, n in enumerate(sizes)]
    g, batch, _, _ = build(systems, prec)
    off = np.insert(batch.atom_offset, 3, batch.atom_offset[3]).astype(np.int32)   # an empty system
    plan = g.Plan(off, prec)
    atoms = g.Atoms.from_batch(plan, batch)
    p = params_pair()[0]
    first = g.evaluate(plan, atoms, p)
    for _ in range(3):
        again = g.evaluate(plan, atoms, p)
        g.radii(plan, atoms, p)
        alone = g.energy_forces(plan, atoms, p, force=False, dEdq=False, dEdrho=False)
        for k in ("e_coul", "e_gb"):
            assert torch.equal(first[k], again[k]) and torch.equal(first[k], alone[k])
    E = (first["e_coul"] + first["e_gb"]).cpu().numpy()
    w = np.append(0.5 * batch.q * first["dEdq"].double().cpu().numpy(), 0.0)
    scale = first["e_coul"].abs().cpu().numpy() + first["e_gb"].abs().cpu().numpy()
    for b in range(len(off) - 1):
        # each atom's 1/2 q dE/dq is rounded like the pair sums it is made of
        half = w[off[b]:off[b + 1]]
        assert abs(E[b] - half.sum()) <= tol * max(scale[b], np.abs(half).sum()), b
    assert E[3] == 0.0


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_energy_sums_of_small_systems(prec):
    # systems of up to 256 atoms are summed a wavefront each: the same values, bit for
    # bit, as beside a system of 257, where each has a workgroup; from every launch that
    # sums them
    sizes = [1, 256, 63, 64, 65, 255, 128, 2]
    systems = [synth.make_system(160 + k, n, 18.0 * (max(n, 8) / 2500.0) ** (1 / 3)) for k, n in enumerate(sizes)]
    large = synth.make_system(170, 257, 18.0 * (257 / 2500.0) ** (1 / 3))
    p, got = params_pair()[0], []
    for batch_systems in (systems, systems + [large]):
        for kw in ({}, {"j_blocks": 1}):
            g, batch, _, atoms = build(batch_systems, prec)
            off = np.insert(batch.atom_offset, 3, batch.atom_offset[3]).astype(np.int32)   # an empty system
            plan = g.Plan(off, prec, j_blocks_per_item=kw.get("j_blocks"))
            for single in (False, True):
                plan.set_single_launch(single)
                full = g.evaluate(plan, atoms, p)
                few = g.evaluate(plan, atoms, p, force=False, dEdq=False, dEdrho=False)
                for out in (full, few):
                    got.append(torch.stack([out["e_coul"][:9], out["e_gb"][:9]]))
    assert got[0][0, 3] == 0.0 and got[0][1, 3] == 0.0 and bool((got[0][1, 1:3] != 0.0).all())
    for other in got[1:]:
        assert torch.equal(got[0], other)
