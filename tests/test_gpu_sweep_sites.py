"""The sequential sweep on site tables at the edges of its kernels, against the
oracle: sites of 1, 2, 3, 63, 64, 255 and 256 atoms (the pairs of one site are
enumerated from a folded triangle, odd and even), a system with no sites, and a
system of 70 sites, more than the couplings a workgroup keeps on chip.  FP64
plan: Delta G of every visit at 1e-9 relative, decisions, states and charges
equal (no uniform lies within 1e-9 of its acceptance probability)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_common import build, params_pair

pytestmark = pytest.mark.gpu


def _with_sites(seed, n, sizes):
    s = synth.make_system(seed, n, 18.0 * (n / 2500.0) ** (1 / 3))
    rng = np.random.default_rng(seed)
    taken = np.zeros(n, dtype=bool)
    xyz = s.coords()
    for k, size in enumerate(sizes):
        atoms = synth._pick_site_atoms(rng, xyz, taken, size, 18.0)
        make = synth._redox_site if k % 3 == 2 else synth._prot_site
        s.sites.append(make(rng, s.q, atoms))
    synth._apply_states(s)
    return s


@pytest.mark.parametrize("kinds", [3, 1])
def test_sweep_site_sizes_and_counts(kinds):
    systems = [_with_sites(170, 1000, [1, 2, 3, 63, 64, 255, 256]), synth.make_system(171, 100, 6.2),
               _with_sites(172, 900, [1 + k % 3 for k in range(70)])]
    p_gpu, p_or = params_pair()
    g, batch, plan, atoms = build(systems, "fp64")
    rng = np.random.default_rng(5)
    gref = rng.normal(0.0, 1.0, batch.state_count.size)
    # every proposal near balance at the starting charges, so that some are accepted
    g0 = 0
    E = np.array([-0.3, -0.25, -0.2])
    for b, s in enumerate(systems):
        tab = oracle.SiteTables(s)
        dE = oracle.site_dE(s, oracle.radii(s, p_or)["R"], p_or, tables=tab) if s.sites else []
        c = 0
        for site in s.sites:
            for t in range(site.n_states):
                if t != site.state:
                    drive = (1.98720426e-3 * 300.0 * np.log(10) * 7.0 if site.kind == 0 else 23.0605478 * E[b])
                    gref[g0 + t] = gref[g0 + site.state] + dE[c] + rng.normal(0.0, 0.5) \
                        + drive * (site.counts[t] - site.counts[site.state])
                    c += 1
            g0 += site.n_states
    sites = g.Sites.from_batch(plan, batch, gref)
    cur = torch.as_tensor(batch.current_state, device=plan.device)
    u = synth.uniforms(77, (batch.n_sites, 3))
    g.radii(plan, atoms, p_gpu)
    out = g.mc_sweep(plan, sites, atoms, cur, 7.0, E, torch.as_tensor(u, device=plan.device), 300.0, p_gpu,
                     kinds=kinds)
    dG, acc, q = out["dG"].cpu().numpy(), out["accepted"].cpu().numpy(), atoms.q.cpu().numpy()
    m = g0 = n_acc = 0
    for b, s in enumerate(systems):
        ns, n_st = len(s.sites), sum(site.n_states for site in s.sites)
        tab = oracle.SiteTables(s, gref[g0:g0 + n_st])
        if ns:
            q_or, acc_or, dG_or = oracle.mc_sweep(s, oracle.radii(s, p_or)["R"], tab, 7.0, E[b], 300.0,
                                                  u[m:m + ns], kinds, p_or)
            for k in range(ns):
                assert acc[m + k] == acc_or[k], (b, k)
                if acc_or[k] >= 0:
                    assert abs(dG[m + k] - dG_or[k]) <= 1e-9 * max(1.0, abs(dG_or[k])), (b, k)
            assert list(cur.cpu().numpy()[m:m + ns]) == list(tab.current_state)
            assert np.array_equal(q[batch.atom_offset[b]:batch.atom_offset[b + 1]], q_or)
            n_acc += int((acc_or > 0).sum())
        m += ns
        g0 += n_st
    assert n_acc > 0                    # the couplings of accepted visits were used
