"""GPU parity of the cutoff passes on each kind of tile: descreening radii at
which the fits of the part of a ball beyond the sphere hold on every tile, on
some (their domain, S <= 0.18 rgbmax, ends between the blocks' largest S) and
on none, and at which a sphere is smaller than an intrinsic radius; in both
plans, with whole and ragged blocks, touching and separated ones."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_common import TOL, build, compare_system, params_pair, gpu_eval, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("rgbmax", [1.5, 5.0, 8.6, 9.4, 10.0, 14.0, 40.0])
def test_descreening_sphere_sizes(prec, rgbmax):
    systems = [synth.make_system(140, 129, 7.0), synth.make_system(141, 641, 11.5),
               synth.make_system(142, 64, 5.0)]
    # blocks of small balls beside blocks of large ones: the domain of the fits
    # ends inside the batch for rgbmax between 8 and 10
    s = systems[1]
    o = np.argsort(s.screen * (s.rho - 0.09), kind="stable")
    for k in ("x", "y", "z", "q", "rho", "screen"):
        setattr(s, k, getattr(s, k)[o].copy())
    p_gpu, p_or = params_pair()
    p_gpu, p_or = (dataclasses.replace(p, rgbmax=rgbmax) for p in (p_gpu, p_or))
    g, batch, plan, atoms = build(systems, prec)
    res = gpu_eval(plan, atoms, p_gpu)
    for b, s in enumerate(systems):
        compare_system(res, b, batch.atom_offset, oracle.energy_forces(s, p_or), prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("apart", [0, 70])
def test_ball_through_the_other_centre(prec, swap, apart):
    # an atom at the surface of its neighbour's ball (r equal to S_j: 1 - y is zero in
    # that direction, which takes the closed form) while its own ball, small and far
    # from the neighbour's radius, takes the polynomial form.  rho - offset and S are
    # exact in both precisions: rt 0.5 and S 0.25 against rt 1 and S 2 at r 2.  `apart` atoms
    # between them in the list put the pair into a tile off the diagonal.
    rng = np.random.default_rng(0)
    small, large = (0.0, 1.0, 0.5), (2.0, 1.5, 2.0)     # x, rho, screen
    first, last = (large, small) if swap else (small, large)
    t = np.arange(apart)
    cols = [(a, m, b) for a, m, b in zip(first, (1.0 + t % 2, 1.0 + 0 * t, 0.5 + 0 * t), last)]
    x, rho, screen = (np.concatenate([[a], m, [b]]) for a, m, b in cols)
    y = np.concatenate([[0.0], 3.0 + 0.75 * t, [0.0]])
    q = rng.normal(0.0, 0.3, x.size)
    s = synth.System(x, y, np.zeros(x.size), q, rho, screen)
    for k in ("x", "y", "z", "q", "rho", "screen"):
        setattr(s, k, synth.f32(getattr(s, k)))
    p_gpu, p_or = (dataclasses.replace(p, offset=0.5, rgbmax=16.0) for p in params_pair())
    g, batch, plan, atoms = build([s], prec)
    res = gpu_eval(plan, atoms, p_gpu)
    assert not g.check_overflow(plan)
    # (the energies of two small charges, 0.7 kcal/mol, hold 2^-32 kcal/mol: not compared)
    ref = oracle.energy_forces(s, p_or)
    assert np.max(np.abs(res["R"] - ref["R"]) / ref["R"]) <= TOL[prec]["R"]
    for k, r in (("force", "F"), ("dEdq", "phi"), ("dEdrho", "dEdrho")):
        assert rel_inf(res[k], ref[r]) <= TOL[prec]["grad"], k
