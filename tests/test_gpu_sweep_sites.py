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


def _sweep(g, systems, gref, u, E, kinds, p, prec="fp64", T=300.0):
    g, batch, plan, atoms = build(systems, prec)
    sites = g.Sites.from_batch(plan, batch, gref)
    cur = torch.as_tensor(batch.current_state, device=plan.device)
    g.radii(plan, atoms, p)
    out = g.mc_sweep(plan, sites, atoms, cur, 7.0, E, torch.as_tensor(u, device=plan.device), T, p, kinds=kinds)
    return batch, out, cur, atoms.q


@pytest.mark.parametrize("kinds", [3, 2])
def test_sweep_with_couplings_formed_at_the_visits(kinds):
    # more pairs of sites than are formed before the first decision, 363,548: systems of
    # 600 sites of one atom, 500 of two and 340 of three, one whose sites have up to
    # 256 atoms, and one without sites, against the oracle
    systems = [_with_sites(173, 700, [1] * 600), synth.make_system(171, 100, 6.2),
               _with_sites(174, 1100, [2] * 500), _with_sites(175, 1000, [1, 2, 3, 63, 64, 255, 256]),
               _with_sites(176, 1100, [3] * 340)]
    p_gpu, p_or = params_pair()
    T, E = 300.0, np.array([-0.3, -0.25, -0.2, -0.25, -0.3])
    rng = np.random.default_rng(6)
    n_st = [sum(site.n_states for site in s.sites) for s in systems]
    gref = np.zeros(sum(n_st))
    Rs = [oracle.radii(s, p_or)["R"] for s in systems]
    g0 = 0
    for s, R, e in zip(systems, Rs, E):             # every proposal near balance at the start
        dE = oracle.site_dE(s, R, p_or, tables=oracle.SiteTables(s)) if s.sites else []
        c = 0
        for site in s.sites:
            drive = 1.98720426e-3 * T * np.log(10) * 7.0 if site.kind == 0 else 23.0605478 * e
            for t in range(site.n_states):
                if t != site.state:
                    gref[g0 + t] = dE[c] + rng.normal(0.0, 0.5) + drive * (site.counts[t] - site.counts[site.state])
                    c += 1
            g0 += site.n_states
    u = synth.uniforms(78, (sum(len(s.sites) for s in systems), 3))
    from gpu_common import gb
    batch, out, cur, q = _sweep(gb(), systems, gref, u, E, kinds, p_gpu)
    dG, acc, ne = (out[k].cpu().numpy() for k in ("dG", "accepted", "n_electrons"))
    q, cur = q.cpu().numpy(), cur.cpu().numpy()
    m = g0 = n_acc = 0
    for b, s in enumerate(systems):
        ns = len(s.sites)
        q_or = np.asarray(s.q, dtype=np.float64)
        if ns:
            tab = oracle.SiteTables(s, gref[g0:g0 + n_st[b]])
            q_or, acc_or, dG_or = oracle.mc_sweep(s, Rs[b], tab, 7.0, E[b], T, u[m:m + ns], kinds, p_or)
            assert np.array_equal(acc[m:m + ns], acc_or), b
            on = acc_or >= 0
            assert np.all(np.abs(dG[m:m + ns] - dG_or)[on] <= 1e-9 * np.maximum(1.0, np.abs(dG_or[on]))), b
            assert np.array_equal(cur[m:m + ns], tab.current_state)
            n_acc += int((acc_or > 0).sum())
            assert ne[b] == sum(site.counts[k] for site, k in zip(s.sites, tab.current_state) if site.kind == 1)
        assert np.array_equal(q[batch.atom_offset[b]:batch.atom_offset[b + 1]], q_or)
        m += ns
        g0 += n_st[b]
    assert n_acc > 0                    # the rows of accepted visits were used


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_replicas_of_a_system_at_the_limit_sweep_alike(prec):
    # 1,024 sites of one atom: 16 replicas (8,396,800 pairs of sites) give what one gives
    from gpu_common import gb
    s = _with_sites(177, 1100, [1] * 1024)
    u = synth.uniforms(79, (1024, 3))
    n_st = sum(site.n_states for site in s.sites)
    p = params_pair()[0]
    _, one, cur1, q1 = _sweep(gb(), [s], np.zeros(n_st), u, -0.2, 3, p, prec, T=3000.0)
    _, all_, cur, q = _sweep(gb(), [s] * 16, np.zeros(16 * n_st), np.tile(u, (16, 1)), -0.2, 3, p, prec, T=3000.0)
    assert 0 < int((one["accepted"] > 0).sum()) < 1024
    for a, b in ((one["accepted"], all_["accepted"]), (one["dG"], all_["dG"]), (cur1, cur), (q1, q)):
        assert torch.equal(a.repeat(16), b)
