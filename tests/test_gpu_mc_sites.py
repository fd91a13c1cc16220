"""The attempt pair on systems with sites of both kinds, of one and of none, and
with sites of 1, 64, 255 and 256 atoms (the most a site may have), against the
oracle: FP64 plan, several attempts from the states the ones before left.  Delta G
at 1e-9 relative, decisions, states, charges, counters and electron counts equal
(no uniform lies within 1e-9 of its acceptance probability)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_common import build, params_pair

pytestmark = pytest.mark.gpu

# (kind, atoms) of each system's sites: 0 protonation, 1 redox
SITES = [[(0, 256), (1, 255), (0, 1)], [(0, 64), (0, 65)], [(1, 256)], [], [(1, 1), (0, 255), (1, 64)]]


def _systems():
    out = []
    for b, sites in enumerate(SITES):
        s = synth.make_system(210 + b, 700, 11.8)
        rng = np.random.default_rng(b)
        taken = np.zeros(s.n, dtype=bool)
        for kind, size in sites:
            atoms = synth._pick_site_atoms(rng, s.coords(), taken, size, 11.8)
            s.sites.append((synth._redox_site if kind else synth._prot_site)(rng, s.q, atoms))
        synth._apply_states(s)
        out.append(s)
    return out


@pytest.mark.parametrize("T", [300.0, 3000.0])
def test_attempts_on_missing_kinds_and_large_sites(T):
    systems = _systems()
    p_gpu, p_or = params_pair()
    g, batch, plan, atoms = build(systems, "fp64")
    B = len(systems)
    rng = np.random.default_rng(3)
    pH, E = rng.uniform(5, 9, B), rng.uniform(-0.3, -0.1, B)
    # every change near balance at the starting charges, so that some are accepted
    gref = np.zeros(batch.state_count.size)
    g0, tabs, qs, Rs, counts = 0, [], [], [], []
    for b, s in enumerate(systems):
        R = oracle.radii(s, p_or)["R"]
        dE = oracle.site_dE(s, R, p_or, tables=oracle.SiteTables(s)) if s.sites else []
        c, first = 0, g0
        for site in s.sites:
            for t in range(site.n_states):
                if t != site.state:
                    drive = (1.98720426e-3 * T * np.log(10) * pH[b] if site.kind == 0
                             else 23.0605478 * E[b])
                    gref[g0 + t] = gref[g0 + site.state] + dE[c] \
                        + drive * (site.counts[t] - site.counts[site.state]) + rng.normal(0.0, 0.3)
                    c += 1
            g0 += site.n_states
        tabs.append(oracle.SiteTables(s, gref[first:g0]) if s.sites else None)
        qs.append(np.asarray(s.q, dtype=np.float64))
        Rs.append(R)
    sites = g.Sites.from_batch(plan, batch, gref)
    cur = torch.as_tensor(batch.current_state, device=plan.device)
    counters = torch.zeros((batch.n_sites, 2), dtype=torch.int64, device=plan.device)
    g.radii(plan, atoms, p_gpu)
    n_acc = both = 0
    for it in range(6):
        u = synth.uniforms(900 + it, (B, 6))
        dE, dG = g.mc_state_dE(plan, sites, atoms, cur, pH, E, T, p_gpu)
        out = g.mc_step(plan, sites, atoms, cur, pH, E, dE, dG, torch.as_tensor(u, device=plan.device), T,
                        p_gpu, counters=counters)
        acc, q = out["accepted"].cpu().numpy(), atoms.q.cpu().numpy()
        st, ne = cur.cpu().numpy(), out["n_electrons"].cpu().numpy()
        m0 = 0
        for b, s in enumerate(systems):
            a0, a1 = batch.atom_offset[b], batch.atom_offset[b + 1]
            if not s.sites:
                assert not acc[b].any() and ne[b] == 0
                assert np.array_equal(q[a0:a1], qs[b])
                continue
            qs[b], o, _ = oracle.mc_step(s, Rs[b], tabs[b], pH[b], E[b], T, u[b], p_or, q=qs[b])
            assert np.array_equal(acc[b], o[:2]), (it, b)
            n = len(s.sites)
            assert np.array_equal(st[m0:m0 + n], tabs[b].current_state)
            assert np.array_equal(q[a0:a1], qs[b])
            want = sum(site.counts[k] for site, k in zip(s.sites, tabs[b].current_state) if site.kind == 1)
            assert ne[b] == want
            n_acc += int(acc[b].sum())
            both += int(acc[b].all())
            m0 += n
    assert n_acc > 0 and both > 0
    total = counters.cpu().numpy().sum(0)
    tried = 6 * sum((any(k == 0 for k, _ in v)) + (any(k == 1 for k, _ in v)) for v in SITES)
    assert total[0] == tried and total[1] == n_acc


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kappa", [0.0, 0.1])
def test_undefined_distance_raises_the_flag(prec, kappa):
    # a coordinate that is not a number: the potential rows raise the flag by themselves,
    # after the one that the radii raised has been read (which clears it)
    s = synth.make_system(216, 300, 9.0, n_redox=1, n_prot=1)
    far = [a for a in range(s.n) if all(a not in site.atoms for site in s.sites)]
    s.y[far[0]] = np.nan
    p = dataclasses.replace(params_pair()[0], kappa=kappa)
    g, batch, plan, atoms = build([s], prec)
    sites = g.Sites.from_batch(plan, batch)
    cur = torch.as_tensor(batch.current_state, device=plan.device)
    g.radii(plan, atoms, p)
    assert g.check_overflow(plan) and not g.check_overflow(plan)
    g.mc_state_dE(plan, sites, atoms, cur, 7.0, -0.2, 300.0, p)
    assert g.check_overflow(plan)
