"""ReplicaMD.run builds its calls' argument lists once, from raw addresses: every
tensor behind them has to stay alive, at its address, through the last call, whatever the
attempts and exchanges of the run allocate.  On the CPU, with the library calls
replaced by recorders."""
import weakref
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_1803_09652_amd import api, runtime

B, N = 2, 5
OUTPUTS = ("R", "e_coul", "e_gb", "force")


class Library:
    """Records, at each call, which of the outputs are alive."""

    def __init__(self):
        self.live, self.calls = {}, []

    def _call(self, name):
        def f(*args):
            given = {a.value for a in args if hasattr(a, "value")}
            alive = {k: r() for k, r in self.live.items()}
            used = {"gb_radii": ("R",), "gb_energy_forces": ("e_coul", "e_gb", "force"),
                    "gb_evaluate": OUTPUTS, "md_langevin_step": ("force",)}[name]
            self.calls.append((name, all(alive[k] is not None and alive[k].data_ptr() in given
                                         for k in used)))
            return 0
        return f

    def __getattr__(self, name):
        return self._call(name)


@pytest.mark.parametrize("single_launch", [False, True])
@pytest.mark.parametrize("attempt_every,exchange_every", [(0, 0), (1, 0), (2, 3), (3, 1)])
def test_outputs_live_until_the_last_call(monkeypatch, single_launch, attempt_every, exchange_every):
    lib = Library()
    outputs = api._eval_outputs

    def tracked(*a):
        out = outputs(*a)
        lib.live = {k: weakref.ref(out[k]) for k in OUTPUTS}
        return out
    cpu = torch.device("cpu")
    monkeypatch.setattr(runtime.L, "load", lambda: lib)
    monkeypatch.setattr(api, "_eval_outputs", tracked)
    monkeypatch.setattr(api, "_stream", lambda dev: None)
    monkeypatch.setattr(api, "mc_state_dE", lambda *a, **k: (torch.zeros(2), torch.zeros(2)))
    monkeypatch.setattr(api, "mc_step", lambda *a, **k: {
        "n_electrons": torch.zeros(B, dtype=torch.int32), "accepted": torch.zeros(B, 2)})
    monkeypatch.setattr(api, "remd_exchange", lambda *a, **k: (torch.zeros(1, dtype=torch.int32), None))
    plan = SimpleNamespace(device=cpu, dtype=torch.float32, n_systems=B, n_atoms=N, handle=None,
                           workspace=torch.zeros(256, dtype=torch.uint8), single_launch=single_launch)
    sites = SimpleNamespace(n_sites=0, site_kind=[], site_system=[])
    v = torch.zeros(N)
    atoms = SimpleNamespace(x=v, y=v, z=v, c=lambda: api.L.gbmc_atoms())
    loop = runtime.ReplicaMD(plan, sites, atoms, [], np.ones(N), np.zeros((3, N)), 7.0, np.zeros(B),
                             attempt_every=attempt_every, exchange_every=exchange_every)
    for n in (1, 6):                                    # a run of its own, and one that follows it
        lib.calls.clear()
        loop.run(n)
        assert sum(name == "md_langevin_step" for name, _ in lib.calls) == n
        assert all(ok for _, ok in lib.calls), lib.calls
