"""The launch search against a stand-in for the library whose times depend on a launch
setting only where the library's do: in rounds that are launches (CPU only)."""
import os
import re
import types

import pytest
import torch

from paper_2308_08410_amd import autotune

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BEST = dict(lanes=8, sweep_blocks=768, sync_batch=32, split=0)


class Lib(types.SimpleNamespace):
    def __init__(self, solver="exact"):
        super().__init__(launch=None, split=1, hold=(0.0, 0, 0), solver=solver, levels=set(), calls=0)

    def set_warm_order(self, plan, on): pass
    def set_queue_split(self, plan, split): self.split = split
    def get_hold(self, plan): return self.hold
    def get_local_solver(self, plan): return dict(solver=self.solver)
    def last_counts(self, plan): return dict(rounds=10, levels=20)
    def eikonal_backward(self, *a, **k): pass

    def set_hold(self, plan, delta, window=0, open_below=0):
        self.hold = (delta, window, open_below)

    def set_launch(self, plan, lanes, sweep_blocks, level_blocks, sync_batch):
        self.launch = dict(lanes=lanes, sweep_blocks=sweep_blocks, sync_batch=sync_batch)
        self.levels.add(level_blocks)

    def get_launch(self, plan):
        return self.launch

    def eikonal_forward(self, plan, *a, out=None, **k):
        out.copy_(torch.linspace(0, 40, out.numel()))
        self.calls += 1
        one_launch = plan.n_v <= 1 << 18 and self.hold[0] <= 0 and self.solver == "exact"
        set_to = dict(self.launch, split=self.split) if self.launch else {}
        off = sum(set_to.get(k) != v for k, v in BEST.items())
        self.ms = 3.0 - 1e-4 * self.calls if one_launch else 4.0 + off - 2.0 * (self.hold[0] == 8.0)


@pytest.mark.parametrize("n_v,solver", [(5000, "exact"), (1 << 18, "exact"), ((1 << 18) + 1, "exact"), (5000, "fista")])
def test_search_finds_what_acts(n_v, solver, monkeypatch):
    lib = Lib(solver)
    monkeypatch.setattr(autotune, "B", lib)

    def time(fn, repeats):
        fn()
        return lib.ms

    monkeypatch.setattr(autotune, "_time", time)
    plan, D = types.SimpleNamespace(n_v=n_v, n_e=6 * n_v), torch.zeros(1)
    rec = autotune.tune(plan, D, None, None, None, use_cache=False, save=False)
    assert {k: rec[k] for k in BEST} == BEST and lib.launch == {k: v for k, v in BEST.items() if k != "split"}
    assert lib.split == BEST["split"] and lib.levels == {2048}
    # a width of twice the mean advance (40 / 10 rounds) is the fastest hold-back of all
    assert rec["hold_delta"] == 8.0 and lib.hold[0] == 8.0 and rec["ms"] == 2.0
    lib = Lib(solver)
    monkeypatch.setattr(autotune, "B", lib)
    rec = autotune.tune(plan, D, None, None, None, use_cache=False, save=False, hold=False)
    assert {k: rec[k] for k in BEST} == BEST and rec["hold_delta"] == 0.0 and lib.hold[0] == 0.0
    assert rec["ms"] < 3.0 if n_v <= 1 << 18 and solver == "exact" else rec["ms"] == 4.0


def test_one_launch_limit_is_the_librarys():
    with open(os.path.join(ROOT, "paper_2308_08410_amd", "csrc", "gbp_internal.h")) as f:
        m = re.search(r"kRoundsTeamVerts = 1 << (\d+);", f.read())
    assert autotune.ONE_LAUNCH_VERTS == 1 << int(m.group(1))
