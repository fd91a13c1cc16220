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
