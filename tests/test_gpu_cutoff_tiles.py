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
from gpu_common import build, compare_system, params_pair, gpu_eval

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
