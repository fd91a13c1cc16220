"""Workloads of the framework as its users run it, with the work each cannot do
without and its result in 64 bits.

Every case is a plain dict.  ``kind`` says which calls one pass makes:

    eval      evaluate(): Born radii, both energies, forces, dE/dq, dE/drho
    energies  radii() + energy_forces() without gradients (rescoring snapshots)
    forces    radii() + energy_forces() for the forces alone (a dynamics step)
    grad      GBEnergy forward and backward (energies as a torch loss)
    step      evaluate(), then one Monte Carlo attempt pair per replica at the
              same coordinates and one exchange attempt along the ladder
    sweep     radii() + mc_sweep(): every site of every system attempted once
    md        ReplicaMD.run(): a few dynamics steps with one attempt pair and
              one exchange attempt

``n_sys`` systems of ``n_min`` .. ``n_max`` atoms (drawn from ``layout``) form
the batch; ``order`` is the plan's processing order (compact blocks, Morton, or
the order in which the atoms came); the remaining keys are the options of the
call.  Systems are globules of the density, charges, radii and screening
factors of the repository's own workloads.
"""
import math

import numpy as np
import torch

import paper_1803_09652_amd as gb
from paper_1803_09652_amd.runtime import ReplicaMD

KB = 1.98720426e-3          # kcal/(mol K)
FARADAY = 23.0605478        # kcal/(mol V)
AKMA = 418.4                # kcal/(mol A amu) -> A/ps^2
T_KELVIN = 300.0
DENSITY = 2500.0 / (4.0 / 3.0 * math.pi * 18.0 ** 3)     # atoms / A^3 of the 2,500-atom globule
K_RESTR = 2000.0            # kcal/mol/A^2, the repository's dynamics restraint
MD_STEPS = 5                # 10 fs between attempts at 2 fs per step
PAIRS_MAX = 4.2e9           # pairs of the largest listed batch


def _case(name, kind, n_sys, n_min, n_max, precision="fp32", order="blocks", kappa=0.0, rgbmax=0.0,
          cutoff=0.0, layout=0, redox=0, prot=0):
    c = {"kind": kind, "n_sys": n_sys, "n_min": n_min, "n_max": n_max, "precision": precision,
         "order": order, "kappa": kappa, "rgbmax": rgbmax, "cutoff": cutoff, "layout": layout,
         "redox": redox, "prot": prot}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small solute in implicit solvent, as a script evaluates it: launches and latency count
        _case("globule_256", "eval", 1, 256, 256, order="input"),
        # the published implicit-solvent setting: 16 replicas of a 237-atom heme peptide, one
        # redox and two propionate sites; ten femtoseconds of dynamics with attempt and exchange
        _case("md_16x237", "md", 16, 237, 237, redox=1, prot=2),
        # the replica-exchange batch of the benchmark: 16 replicas of a 2,500-atom protein,
        # a full evaluation, every candidate state change, the attempts and the exchange
        _case("step_16x2500", "step", 16, 2500, 2500, redox=4, prot=4),
        # the headline batch: 64 proteins of uneven size, everything the evaluation gives
        _case("eval_uneven_64", "eval", 64, 1024, 19488, layout=4),
        # the same batch layout in miniature with odd sizes and 0.1/A of salt
        _case("salt_ragged_24", "eval", 24, 65, 3777, kappa=0.1, layout=5),
        # the double-precision plan on the replica batch
        _case("fp64_16x2500", "eval", 16, 2500, 2500, precision="fp64"),
        # the double-precision plan on one odd-sized protein: reference runs of single systems
        _case("fp64_9973", "eval", 1, 9973, 9973, precision="fp64"),
        # dynamics of a large complex with the descreening and pair cutoffs
        _case("cutoff_100000", "forces", 1, 100000, 100000, rgbmax=15.0, cutoff=16.0),
        # the energies as a differentiable loss: forward and backward on a 10,000-atom protein
        _case("grad_10000", "grad", 1, 10000, 10000),
        # rescoring of 32 snapshots: energies only
        _case("energies_32x4001", "energies", 32, 4001, 4001),
        # a sequential sweep over all sites of all replicas
        _case("sweep_16x2500", "sweep", 16, 2500, 2500, redox=4, prot=4),
        # dynamics forces of one mid-sized protein: a launch that does not fill the chip by far
        _case("forces_1x3001", "forces", 1, 3001, 3001),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "forces", "energies", "grad", "step", "sweep", "md", "cutoff"])
    layout = rng.randrange(1 << 20)
    precision = "fp64" if rng.random() < 0.25 else "fp32"
    order = rng.choice(["blocks", "blocks", "blocks", "morton", "input"])
    kappa = rng.choice([0.0, 0.0, 0.0, 0.05, 0.1, 0.13])
    if kind == "cutoff":
        n = _log_int(rng, 8000, 100000)
        return _case(None, "forces", 1, n, n, precision=precision if n < 40000 else "fp32",
                     order=rng.choice(["blocks", "morton"]), kappa=kappa,
                     rgbmax=rng.choice([12.0, 15.0, 18.0, 25.0]), cutoff=rng.choice([14.0, 16.0, 20.0]),
                     layout=layout)
    if kind in ("step", "sweep", "md"):
        n = _log_int(rng, 230, 800 if kind == "md" else 4000)
        return _case(None, kind, rng.choice([2, 4, 8, 12, 16, 24]), n, n, precision=precision, order=order,
                     kappa=kappa, layout=layout, redox=1 + (n > 800) * rng.randrange(3),
                     prot=1 + rng.randrange(2 + (n > 800) * 4))
    if kind == "grad":
        n = _log_int(rng, 200, 16000)
        return _case(None, kind, 1, n, n, precision=precision, order=order, kappa=kappa, layout=layout)
    n_sys = _log_int(rng, 1, 64)
    # largest system: at most 20,000 atoms, and the batch's pairs below those of the largest
    # listed case (a double-precision pair costs about three times a single-precision one)
    pairs = PAIRS_MAX / (3.5 if precision == "fp64" else 1.0)
    top = min(20000, int(math.sqrt(2.0 * pairs / n_sys)))
    n_max = _log_int(rng, 100, top)
    n_min = n_max if rng.random() < 0.4 else _log_int(rng, max(2, n_max // 12), n_max)
    return _case(None, kind, n_sys, n_min, n_max, precision=precision, order=order, kappa=kappa, layout=layout)


# ---------------------------------------------------------------- inputs

def _sizes(case):
    rng = np.random.default_rng(case["layout"])
    n = rng.integers(case["n_min"], case["n_max"] + 1, size=case["n_sys"])
    n[0], n[-1] = case["n_min"], case["n_max"]
    return n


def _globule(rng, n):
    """n points of a jittered cubic lattice inside a ball of the workloads'
    density (no two closer than about 0.9 A), in random order."""
    a = DENSITY ** (-1.0 / 3.0)
    half = int(math.ceil((3.0 * n / (4.0 * math.pi)) ** (1.0 / 3.0))) + 2
    g = np.arange(-half, half + 1)
    xyz = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3) + rng.uniform(-0.5, 0.5, size=3)
    keep = np.argpartition((xyz ** 2).sum(1), n - 1)[:n]
    xyz = a * xyz[keep] + rng.uniform(-0.62, 0.62, size=(n, 3))
    return xyz[rng.permutation(n)]


def _inputs(case, seed):
    """Host arrays of one batch (values representable in single precision)."""
    rng = np.random.default_rng([seed, case["layout"]])
    off = np.concatenate([[0], np.cumsum(_sizes(case))]).astype(np.int32)
    n = int(off[-1])
    xyz = np.concatenate([_globule(rng, int(m)) for m in np.diff(off)])
    q = rng.normal(0.0, 0.3, size=n)
    q -= np.repeat(np.add.reduceat(q, off[:-1]) / np.diff(off), np.diff(off))
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    d = {"off": off, "xyz": f32(xyz), "q": f32(q), "rho": f32(rng.uniform(1.2, 2.0, n)),
         "screen": f32(rng.uniform(0.7, 0.9, n))}
    if case["redox"] or case["prot"]:
        d["sites"] = _site_tables(case, rng, d)
        B, S = case["n_sys"], len(d["sites"]["site_kind"])
        d["pH"] = np.full(B, 7.0)
        d["E"] = -0.40 + 0.02 * np.arange(B)
        d["u_step"] = rng.random((B, 6))
        d["u_sweep"] = rng.random((S, 3))
        d["u_x"] = rng.random(B)
        d["mass"] = f32(rng.uniform(12.0, 16.0, n))
        d["v"] = f32(rng.standard_normal((3, n)) * np.sqrt(KB * T_KELVIN * AKMA / d["mass"]))
        d["xi"] = f32(rng.standard_normal((MD_STEPS, 3, n)))
    return d


def _site_tables(case, rng, d):
    """Disjoint sites of nearest atoms: redox sites of up to 74 atoms and two
    states, protonation sites of 10 .. 20 atoms and five states."""
    t = {k: [] for k in ("site_system", "site_kind", "site_atoms", "state_charges", "state_count", "state")}
    sao, sso, sco = [0], [0], [0]
    for b in range(case["n_sys"]):
        a0, a1 = int(d["off"][b]), int(d["off"][b + 1])
        free = np.ones(a1 - a0, dtype=bool)
        xyz = d["xyz"][a0:a1]
        for m in range(case["redox"] + case["prot"]):
            kind = 1 if m < case["redox"] else 0
            k = min(74, (a1 - a0) // 3) if kind else int(rng.integers(10, 21))
            idx = np.nonzero(free)[0]
            c = xyz[rng.integers(0, a1 - a0)]
            sel = np.sort(idx[np.argsort(((xyz[idx] - c) ** 2).sum(1), kind="stable")[:k]])
            free[sel] = False
            q0 = d["q"][a0 + sel]
            states = [q0]
            for _ in range(1 if kind else 4):
                dq = rng.normal(0.0, 0.05, size=k)
                states.append(q0 + dq + ((-1.0 if kind else 1.0) - dq.sum()) / k)
            cur = int(rng.integers(0, len(states)))
            states = [s.astype(np.float32).astype(np.float64) for s in states]
            d["q"][a0 + sel] = states[cur]
            t["site_system"].append(b)
            t["site_kind"].append(kind)
            t["site_atoms"].extend((a0 + sel).tolist())
            t["state"].append(cur)
            for s, row in enumerate(states):
                t["state_charges"].extend(row.tolist())
                t["state_count"].append(int(s > 0))
                sco.append(len(t["state_charges"]))
            sao.append(len(t["site_atoms"]))
            sso.append(sso[-1] + len(states))
    t["state_gref"] = rng.normal(0.0, 2.0, size=len(t["state_count"]))
    out = {k: np.asarray(v, dtype=np.float64 if k in ("state_charges", "state_gref") else np.int32)
           for k, v in t.items()}
    out.update(site_atom_offset=np.int32(sao), site_state_offset=np.int32(sso), state_charge_offset=np.int32(sco))
    return out


def prepare(case, seed):
    d = _inputs(case, seed)
    plan = gb.Plan(d["off"], case["precision"])
    x, y, z = (np.ascontiguousarray(d["xyz"][:, k]) for k in range(3))
    if case["order"] != "input":
        plan.set_order((gb.block_order if case["order"] == "blocks" else gb.spatial_order)(d["off"], x, y, z))
    s = {"kind": case["kind"], "plan": plan,
         "atoms": gb.Atoms(plan, x, y, z, d["q"], d["rho"], d["screen"]),
         "params": gb.GBParams(kappa=case["kappa"], rgbmax=case["rgbmax"], cutoff=case["cutoff"])}
    dev = plan.device
    if case["kind"] == "grad":
        t = lambda a: torch.as_tensor(a, dtype=plan.dtype, device=dev)
        s["leaves"] = [t(d["xyz"]).requires_grad_(), t(d["q"]).requires_grad_(), t(d["rho"]).requires_grad_()]
        s["screen"] = t(d["screen"])
    if "sites" in d:
        t = {k: v for k, v in d["sites"].items() if k != "state"}
        s["sites"] = gb.Sites(plan, **t)
        s["state0"] = torch.as_tensor(d["sites"]["state"], device=dev)
        s["state"] = s["state0"].clone()
        s["q_out"] = s["atoms"].q.clone()
        for k in ("pH", "E", "u_step", "u_sweep", "u_x"):
            s[k] = torch.as_tensor(d[k], device=dev)
        s["ladder"] = torch.arange(plan.n_systems, dtype=torch.int32, device=dev)
        s["rep"] = s["ladder"].clone()
    if case["kind"] == "md":
        md = ReplicaMD(plan, s["sites"], s["atoms"], d["sites"]["state"], 1.0 / d["mass"], d["v"], d["pH"],
                       d["E"], attempt_every=MD_STEPS, exchange_every=MD_STEPS, params=s["params"],
                       xref=np.stack([x, y, z]), k_restr=K_RESTR, T=T_KELVIN)
        s["md"] = md
        s["xi"] = torch.as_tensor(d["xi"], dtype=plan.dtype, device=dev)
        s["live"] = [md.atoms.x, md.atoms.y, md.atoms.z, md.atoms.q, md.v, md.state, md.rep_of_rung, md.E_rep]
        s["saved"] = [t.clone() for t in s["live"]]
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------ a pass

def run(s):
    kind, plan, atoms, p = s["kind"], s["plan"], s["atoms"], s["params"]
    if kind == "eval":
        return gb.evaluate(plan, atoms, p)
    if kind == "energies":
        R = gb.radii(plan, atoms, p)
        e = gb.energy_forces(plan, atoms, p, force=False, dEdq=False, dEdrho=False)
        return {"R": R, "e_coul": e["e_coul"], "e_gb": e["e_gb"]}
    if kind == "forces":
        R = gb.radii(plan, atoms, p)
        return {"R": R, "force": gb.energy_forces(plan, atoms, p, dEdq=False, dEdrho=False)["force"]}
    if kind == "grad":
        pos, q, rho = s["leaves"]
        E = gb.GBEnergy.apply(pos, q, rho, s["screen"], plan, p)
        g = torch.autograd.grad(E.sum(), (pos, q, rho))
        return {"E": E.detach(), "pos": g[0], "q": g[1], "rho": g[2]}
    if kind == "step":
        s["state"].copy_(s["state0"])
        s["q_out"].copy_(atoms.q)
        s["rep"].copy_(s["ladder"])
        out = gb.evaluate(plan, atoms, p)
        dE, dG = gb.mc_state_dE(plan, s["sites"], atoms, s["state"], s["pH"], s["E"], T_KELVIN, p)
        mc = gb.mc_step(plan, s["sites"], atoms, s["state"], s["pH"], s["E"], dE, dG, s["u_step"], T_KELVIN, p,
                        q_out=s["q_out"])
        acc, E_rep = gb.remd_exchange(s["E"], mc["n_electrons"], s["rep"], 0, s["u_x"], T_KELVIN)
        out.update(dE=dE, dG=dG, state=s["state"], q=s["q_out"], n_electrons=mc["n_electrons"],
                   accepted=mc["accepted"], exchanged=acc, rep=s["rep"], E_rep=E_rep)
        return out
    if kind == "sweep":
        s["state"].copy_(s["state0"])
        s["q_out"].copy_(atoms.q)
        R = gb.radii(plan, atoms, p)
        out = gb.mc_sweep(plan, s["sites"], atoms, s["state"], s["pH"], s["E"], s["u_sweep"], T_KELVIN, p,
                          q_out=s["q_out"])
        return {"R": R, "state": s["state"], "q": s["q_out"], **out}
    md = s["md"]                                   # the same ten femtoseconds again
    torch._foreach_copy_(s["live"], s["saved"])
    md.step_index = md.n_exchanges = 0
    rec = md.run(MD_STEPS, xi=s["xi"], u_mc=s["u_step"][None], u_x=s["u_x"][None])
    return {"x": md.atoms.x, "y": md.atoms.y, "z": md.atoms.z, "v": md.v, "q": md.atoms.q, "state": md.state,
            "rep": md.rep_of_rung, "E_rep": md.E_rep, "n_electrons": rec["n_electrons"]}


# -------------------------------------------------------- indispensable work

def work(case):
    n = _sizes(case).astype(np.float64)
    N, B, w = float(n.sum()), float(case["n_sys"]), 8.0 if case["precision"] == "fp64" else 4.0
    pairs = float((n * (n - 1) / 2).sum())

    def within(r):
        """Pairs closer than r (0: all): the ball around an atom, cut by the globule's surface."""
        if r <= 0.0:
            return pairs
        a = (3.0 * n / (4.0 * math.pi * DENSITY)) ** (1.0 / 3.0)
        t = np.minimum(r / (2.0 * a), 1.0)
        return float((n * (n - 1) / 2 * np.minimum(1.0, 8 * t ** 3 - 9 * t ** 4 + 2 * t ** 6)).sum())

    # flops per unordered pair, both directions (closed forms): descreening 60,
    # energies alone 24, energies with explicit gradients 54, Born chain 80; salt adds 8
    salt = 8.0 if case["kappa"] else 0.0
    rad, en, gr, ch = 60.0 * within(case["rgbmax"]), 24.0 + salt, 54.0 + salt, 80.0 * within(case["rgbmax"])
    we = within(case["cutoff"])
    full = rad + gr * we + ch
    inp = 6 * w * N
    rows = 0.0
    if case["redox"] or case["prot"]:
        rows = float(((case["redox"] * np.minimum(74, n // 3) + case["prot"] * 15) * n).sum()) * 40.0
    return {
        "eval": lambda: {"bytes": inp + 6 * w * N + 16 * B, "flops": full},
        "energies": lambda: {"bytes": inp + w * N + 16 * B, "flops": rad + en * we},
        "forces": lambda: {"bytes": inp + 4 * w * N, "flops": full},
        "grad": lambda: {"bytes": inp + 5 * w * N + 8 * B, "flops": full},
        "step": lambda: {"bytes": inp + 7 * w * N + 100 * B, "flops": full + rows},
        "sweep": lambda: {"bytes": inp + 2 * w * N + 100 * B, "flops": rad + rows},
        "md": lambda: {"bytes": MD_STEPS * (inp + 22 * w * N), "flops": MD_STEPS * full + rows},
    }[case["kind"]]()


# ------------------------------------------------------------- in 64 bits

class _Exact:
    """The energies of one system and their derivatives, row block by row block
    in double precision, from the definitions."""

    def __init__(self, case, dev):
        self.kC, self.kT, self.kO = 332.0522, 332.0522 * (1.0 - 1.0 / 78.5), 332.0522 / 78.5
        self.kappa, self.rgbmax, self.cutoff = case["kappa"], case["rgbmax"], case["cutoff"]
        self.dev = dev

    @staticmethod
    def _shell(r, L, S, grad):
        """J/(4r), the integral over the part of ball S beyond radius L (and its
        r and S partials at fixed L): J = e - ln(1 + e) + (S - r) e^2 / (2U)."""
        U = r + S
        e = (U - L) / L
        J = e - torch.log1p(e) + (S - r) * e * e / (2 * U)
        if not grad:
            return J / (4 * r)
        eU = e / U
        cross = (S - r) * eU * (1 / L - 0.5 * eU)
        return (eU * (1 - 0.5 * e) + cross - J / r) / (4 * r), (eU * (1 + 0.5 * e) + cross) / (4 * r)

    def hct(self, r, rt, S, grad=False):
        """H (or dH/dr, dH/drt, dH/dS) of balls S at distance r around radii rt."""
        ad = (r - S).abs()
        at_rt = rt > ad
        L = torch.where(at_rt, rt.expand_as(ad), ad)
        eng = rt < S - r
        zero = rt >= r + S
        c = self.rgbmax
        if not grad:
            H = self._shell(r, L, S, False) + torch.where(eng, 1 / rt - 1 / L, 0.0)
            if c > 0:
                H = H - torch.where(r + S > c, self._shell(r, torch.full_like(r, c), S, False), 0.0)
                zero = zero | (r - S >= c) | (rt >= c)
            return torch.where(zero, 0.0, H)
        dr, dS = self._shell(r, L, S, True)
        drt = torch.where(at_rt, ((L - r) ** 2 - S * S) / (4 * r * L ** 3), torch.where(eng, -1 / rt ** 2, 0.0))
        if c > 0:
            cr, cS = self._shell(r, torch.full_like(r, c), S, True)
            st = r + S > c
            dr, dS = dr - torch.where(st, cr, 0.0), dS - torch.where(st, cS, 0.0)
            zero = zero | (r - S >= c) | (rt >= c)
        return tuple(torch.where(zero, 0.0, v) for v in (dr, drt, dS))

    def _blocks(self, xyz):
        n = len(xyz)
        step = max(1, (1 << (25 if self.dev == "cuda" else 21)) // max(n, 1))
        for a in range(0, n, step):
            d = xyz[a:a + step, None, :] - xyz[None, :, :]
            r2 = (d * d).sum(-1)
            own = torch.arange(a, min(a + step, n), device=xyz.device)[:, None] == torch.arange(n, device=xyz.device)
            yield slice(a, min(a + step, n)), d, torch.where(own, 1.0, r2), own

    def radii(self, xyz, rho, screen):
        rt = rho - 0.09
        S = screen * rt
        sums = torch.zeros_like(rho)
        for i, _, r2, own in self._blocks(xyz):
            sums[i] = torch.where(own, 0.0, self.hct(r2.sqrt(), rt[i, None], S[None])).sum(1)
        psi = rt * sums
        th = torch.tanh(psi - 0.8 * psi ** 2 + 4.85 * psi ** 3)
        R = 1 / (1 / rt - th / rho)
        dR = R * R * (1 - th * th) * (1 - 1.6 * psi + 14.55 * psi ** 2) / rho
        return R, dR, sums, th

    def factor(self, f):
        """k d(f) and its slope factor."""
        if self.kappa == 0.0:
            return torch.full_like(f, self.kT), torch.full_like(f, self.kT)
        es = self.kO * torch.exp(-self.kappa * f)
        return self.kC - es, self.kC - es - es * self.kappa * f

    def all(self, xyz, q, rho, screen, grad=True):
        R, dR, sums, th = self.radii(xyz, rho, screen)
        rt = rho - 0.09
        S = screen * rt
        kd, ks = self.factor(R)
        e_c = torch.zeros((), dtype=torch.float64, device=xyz.device)
        e_g = -0.5 * (kd * q * q / R).sum()
        phi = -kd * q / R
        G = 0.5 * ks * q * q / R ** 2
        F = torch.zeros_like(xyz)
        for i, d, r2, own in self._blocks(xyz):
            on = ~own & (r2 < self.cutoff ** 2) if self.cutoff > 0 else ~own
            ir = torch.where(on, r2.rsqrt(), 0.0)
            RR = R[i, None] * R[None]
            D = r2 / (4 * RR)
            ex = torch.exp(-D)
            f = (r2 + RR * ex).sqrt()
            kd, ks = self.factor(f)
            kf = torch.where(on, kd / f, 0.0)
            qq = q[i, None] * q[None]
            e_c += 0.5 * self.kC * (qq * ir).sum()
            e_g -= 0.5 * (qq * kf).sum()
            if not grad:
                continue
            phi[i] += (q[None] * (self.kC * ir - kf)).sum(1)
            w = torch.where(on, ks * qq / f ** 3, 0.0)
            G[i] += 0.5 * (w * ex * (1 + D) * R[None]).sum(1)
            F[i] -= ((w * (1 - 0.25 * ex) - self.kC * qq * ir ** 3)[..., None] * d).sum(1)
        out = {"R": R, "e_coul": e_c, "e_gb": e_g}
        if not grad:
            return out
        B = G * dR
        w = B * rt
        drho = G * R * R * (1 / rt ** 2 - th / rho ** 2) + B * sums
        for i, d, r2, own in self._blocks(xyz):
            r = r2.sqrt()
            a0, a1, _ = self.hct(r, rt[i, None], S[None], True)
            b0, _, b2 = self.hct(r, rt[None].expand_as(r), S[i, None].expand_as(r), True)
            off = lambda v: torch.where(own, 0.0, v)
            F[i] -= ((off(w[i, None] * a0 + w[None] * b0) / r)[..., None] * d).sum(1)
            drho[i] += w[i] * off(a1).sum(1) + screen[i] * off(w[None] * b2).sum(1)
        return dict(out, force=F, dEdq=phi, dEdrho=drho)

    def K(self, xa, Ra, xb, Rb):
        """The charge-charge matrix (self terms on coincident points)."""
        r2 = ((xa[:, None] - xb[None]) ** 2).sum(-1)
        same = r2 == 0.0
        RR = Ra[:, None] * Rb[None]
        f = (r2 + RR * torch.exp(-r2 / (4 * RR))).sqrt()
        k = torch.where(same, 0.0, self.kC * torch.where(same, 1.0, r2).rsqrt()) - self.factor(f)[0] / f
        return torch.where(~same & (r2 >= self.cutoff ** 2), 0.0, k) if self.cutoff > 0 else k


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    n = _sizes(case).astype(np.float64)
    passes = MD_STEPS if case["kind"] == "md" else 1
    if passes * float((n * n).sum()) > (1.3e10 if dev == "cuda" else 3e7):
        return None
    d = _inputs(case, seed)
    x = _Exact(case, dev)
    off = d["off"]
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev)
    xyz, q, rho, screen = t(d["xyz"]), t(d["q"]), t(d["rho"]), t(d["screen"])
    spans = [slice(int(a), int(b)) for a, b in zip(off[:-1], off[1:])]
    kind = case["kind"]

    def batch(grad=True):
        per = [x.all(xyz[b], q[b], rho[b], screen[b], grad) for b in spans]
        return {k: (torch.stack if k.startswith("e_") else torch.cat)([o[k] for o in per]) for k in per[0]}

    if kind == "eval":
        return batch()
    if kind == "energies":
        return batch(False)
    if kind == "forces":
        o = batch()
        return {"R": o["R"], "force": o["force"]}
    if kind == "grad":
        o = batch()
        return {"E": o["e_coul"] + o["e_gb"], "pos": -o["force"], "q": o["dEdq"], "rho": o["dEdrho"]}
    mc = _MonteCarlo(x, d, spans)
    if kind == "sweep":
        R = torch.cat([x.radii(xyz[b], rho[b], screen[b])[0] for b in spans])
        dG = mc.sweep(xyz, R, q, d["E"])
        return {"R": R, "state": None, "q": None, "n_electrons": None, "accepted": None, "dG": t(dG)}
    if kind == "step":
        o = batch()
        dE, dG = mc.candidates(xyz, o["R"], q, d["E"])
        return dict(o, dE=t(dE), dG=t(dG), state=None, q=None, n_electrons=None, accepted=None, exchanged=None,
                    rep=None, E_rep=None)
    # md: leapfrog Langevin steps; the attempt and the exchange precede the last step's forces
    dt, gamma = 0.002, 5.0
    a = 0.5 * gamma * dt
    v, im, xi, ref = t(d["v"]), t((1.0 / d["mass"]).astype(np.float32 if case["precision"] == "fp32" else np.float64)), \
        t(d["xi"]), xyz.clone()
    for k in range(MD_STEPS):
        if k == MD_STEPS - 1:
            R = torch.cat([x.radii(xyz[b], rho[b], screen[b])[0] for b in spans])
            q = mc.attempt(xyz, R, q, d["E"])
        F = torch.cat([x.all(xyz[b], q[b], rho[b], screen[b])["force"] for b in spans]) - K_RESTR * (xyz - ref)
        v = ((1 - a) * v + dt * AKMA * F.T * im + torch.sqrt(2 * gamma * KB * T_KELVIN * dt * AKMA * im) * xi[k]) / (1 + a)
        xyz = xyz + dt * v.T
    return {"x": xyz[:, 0], "y": xyz[:, 1], "z": xyz[:, 2], "v": v, "q": None, "state": None, "rep": None,
            "E_rep": None, "n_electrons": None}


class _MonteCarlo:
    """Candidate energies, the attempt pair and the sweep on given radii."""

    def __init__(self, x, d, spans):
        self.x, self.d, self.spans, self.s = x, d, spans, d["sites"]

    def _site(self, m):
        s = self.s
        atoms = s["site_atoms"][s["site_atom_offset"][m]:s["site_atom_offset"][m + 1]]
        g0, g1 = s["site_state_offset"][m], s["site_state_offset"][m + 1]
        rows = s["state_charges"][s["state_charge_offset"][g0]:s["state_charge_offset"][g1]].reshape(g1 - g0, -1)
        return torch.as_tensor(atoms.astype(np.int64), device=self.x.dev), torch.as_tensor(rows, device=self.x.dev), g0

    def _delta(self, m, cur, new, xyz, R, q, E):
        atoms, rows, g0 = self._site(m)
        b = int(self.s["site_system"][m])
        i = self.spans[b]
        dq = rows[new] - rows[cur]
        phi = self.x.K(xyz[atoms], R[atoms], xyz[i], R[i]) @ q[i]
        de = float(dq @ phi + 0.5 * dq @ (self.x.K(xyz[atoms], R[atoms], xyz[atoms], R[atoms]) @ dq))
        drive = FARADAY * E[b] if self.s["site_kind"][m] else KB * T_KELVIN * math.log(10.0) * self.d["pH"][b]
        c, g = self.s["state_count"], self.s["state_gref"]
        return de, de + drive * float(c[g0 + new] - c[g0 + cur]) - (g[g0 + new] - g[g0 + cur])

    def candidates(self, xyz, R, q, E):
        out = []
        for m, cur in enumerate(self.s["state"]):
            n_states = self.s["site_state_offset"][m + 1] - self.s["site_state_offset"][m]
            out += [self._delta(m, cur, new, xyz, R, q, E) for new in range(n_states) if new != cur]
        return [o[0] for o in out], [o[1] for o in out]

    def _try(self, m, u_state, u_acc, state, xyz, R, q, E):
        n_states = int(self.s["site_state_offset"][m + 1] - self.s["site_state_offset"][m])
        pick = min(int(u_state * (n_states - 1)), n_states - 2)
        new = pick if pick < state[m] else pick + 1
        dg = self._delta(m, state[m], new, xyz, R, q, E)[1]
        if u_acc < math.exp(min(700.0, -dg / (KB * T_KELVIN))):
            atoms, rows, _ = self._site(m)
            q = q.index_copy(0, atoms, rows[new])
            state[m] = new
        return dg, q

    def attempt(self, xyz, R, q, E):
        state = self.s["state"].copy()
        for b in range(len(self.spans)):
            u = self.d["u_step"][b]
            for kind, v in ((0, u[:3]), (1, u[3:])):
                mine = [m for m in range(len(state)) if self.s["site_system"][m] == b and self.s["site_kind"][m] == kind]
                if mine:
                    m = mine[min(int(v[0] * len(mine)), len(mine) - 1)]
                    q = self._try(m, v[1], v[2], state, xyz, R, q, E)[1]
        return q

    def sweep(self, xyz, R, q, E):
        state, u = self.s["state"].copy(), self.d["u_sweep"]
        dG = np.zeros(len(state))
        for kind in (0, 1):
            mine = [m for m in range(len(state)) if self.s["site_kind"][m] == kind]
            for m in sorted(mine, key=lambda k: (self.s["site_system"][k], u[k, 0], k)):
                dG[m], q = self._try(m, u[m, 1], u[m, 2], state, xyz, R, q, E)
        return dG
