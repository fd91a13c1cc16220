"""The work-shape autotuner: its size buckets and cache (CPU), and on the GPU a
sweep over a few candidate shapes that picks one per pass, records it, and
whose shapes give the same results bitwise as the library defaults."""
import numpy as np
import pytest

from paper_1803_09652_amd import autotune as at


def test_bucket_key_groups_batches_by_powers_of_two():
    a = at.bucket_key([0, 2500, 5000], "fp32")
    assert a == at.bucket_key([0, 2400, 4900], "fp32")          # same powers of two
    assert a != at.bucket_key([0, 2500, 5000], "fp64")          # precision is part of the key
    assert a != at.bucket_key([0, 2500, 5000, 7500], "fp32")    # more systems
    assert a != at.bucket_key([0, 5000, 10000], "fp32")         # larger systems
    assert at.bucket_key([0], "fp32").startswith("fp32:")       # empty batch still keys


def test_cache_round_trip(tmp_path, monkeypatch):
    path = tmp_path / "tuning.json"
    monkeypatch.setenv("GBMC_TUNING_CACHE", str(path))
    off = [0, 900, 1233]
    assert at.lookup(off, "fp32") is None
    at._save_cache({at.bucket_key(off, "fp32"): {"j_blocks_per_item": [1, 2, 4],
                                                "waves_per_group": [2, 4, 8], "pair_ms": 1.0}})
    assert at.lookup(off, "fp32") == ((1, 2, 4), (2, 4, 8))
    assert at.lookup(off, "fp64") is None
    path.write_text("not json")
    assert at.lookup(off, "fp32") is None                        # a broken cache is ignored


@pytest.mark.gpu
def test_tune_picks_a_candidate_per_pass_and_keeps_results(tmp_path, monkeypatch):
    import torch
    import synth
    from gpu_common import build, gpu_eval, params_pair
    monkeypatch.setenv("GBMC_TUNING_CACHE", str(tmp_path / "tuning.json"))
    systems = [synth.make_system(31, 700, 10.0), synth.make_system(32, 1500, 14.0)]
    batch = synth.make_batch(systems)
    cands = [(1, 1), (2, 4), (4, 2)]
    r = at.tune(batch, "fp32", candidates=cands, reps=2)
    jbs, wvs = r["best"]
    for k in range(3):
        assert (jbs[k], wvs[k]) in cands
    assert set(r["ms"]) == {f"{j}x{w}" for j, w in cands}
    assert all(v > 0 for v in r["ms"].values())
    # each pass takes its own best shape (medians per kernel, so within noise of any one shape)
    assert r["pair_ms"] <= 1.05 * min(r["ms"].values())
    assert at.lookup(batch.atom_offset, "fp32") == (tuple(jbs), tuple(wvs))
    p_gpu, _ = params_pair()
    _, _, plan_d, atoms_d = build(systems, "fp32")
    _, _, plan_t, atoms_t = build(systems, "fp32", j_blocks=jbs, waves=wvs)
    a, b = gpu_eval(plan_d, atoms_d, p_gpu), gpu_eval(plan_t, atoms_t, p_gpu)
    torch.cuda.synchronize()
    for k in ("R", "Ec", "Egb", "force", "dEdq", "dEdrho"):
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("untuned,best", [(0.5, ((None,) * 3, (None,) * 3)), (2.5, ((1, 2, 1), (4, 1, 2)))])
def test_tune_weighs_the_untuned_plan(tmp_path, monkeypatch, untuned, best):
    # the plan without a shape takes kernels that no shape asks for: it is a candidate
    # of its own, and wins where it is faster than the best shapes together (0.6 each)
    from types import SimpleNamespace
    monkeypatch.setenv("GBMC_TUNING_CACHE", str(tmp_path / "tuning.json"))
    fast = {"radii_pairs": (1, 4), "energy_pairs": (2, 1), "chain_pairs": (1, 2)}

    class Plan:
        def __init__(self, off, prec, j_blocks_per_item=None, waves_per_group=None):
            self.shape = (j_blocks_per_item, waves_per_group)

        def set_timing(self, on):
            pass

        def kernel_ms(self):
            if self.shape == (None, None):
                return {k: untuned for k in at.PAIR_KERNELS}
            return {k: 0.6 if self.shape == s else 1.0 for k, s in fast.items()}
    monkeypatch.setattr(at.api, "Plan", Plan)
    monkeypatch.setattr(at.api, "Atoms", SimpleNamespace(from_batch=lambda plan, batch: None))
    for name in ("radii", "energy_forces"):
        monkeypatch.setattr(at.api, name, lambda *a: None)
    monkeypatch.setattr(at.torch.cuda, "synchronize", lambda: None)
    batch = SimpleNamespace(atom_offset=np.array([0, 256]))
    r = at.tune(batch)
    assert r["best"] == best == at.lookup(batch.atom_offset)
    assert r["pair_ms"] == pytest.approx(min(3 * untuned, 1.8)) and r["ms"]["default"] == pytest.approx(3 * untuned)
    # with a list of candidates the choice stays inside it
    assert at.tune(batch, candidates=[(1, 2)], use_cache=False)["best"] == ((1,) * 3, (2,) * 3)


@pytest.mark.gpu
def test_tuned_small_plan_is_not_slower_than_an_untuned_one(tmp_path, monkeypatch):
    # a triple of None is no shape at all: the tuner's result for a small batch makes the
    # plan that runs one workgroup per item (kernel times of 256 atoms: about half)
    import synth
    from gpu_common import build, gb, params_pair
    monkeypatch.setenv("GBMC_TUNING_CACHE", str(tmp_path / "tuning.json"))
    systems = synth.globule_256()
    batch = synth.make_batch(systems)
    r = at.tune(batch, "fp32", reps=3)
    assert r["best"] == ((None,) * 3, (None,) * 3)
    g, ms = gb(), {}
    for name, (jb, wv) in (("tuned", r["best"]), ("walk", ((1, 1, 1), (2, 4, 4)))):
        _, _, plan, atoms = build(systems, "fp32", j_blocks=jb, waves=wv)
        g.evaluate(plan, atoms, params_pair()[0])
        plan.set_timing(True)
        for _ in range(20):
            g.evaluate(plan, atoms, params_pair()[0])
        ms[name] = sum(plan.kernel_ms().values())
    assert ms["tuned"] < 0.8 * ms["walk"], ms
