"""The autotuner's cache and trials on a stub lattice: a choice cached under the
keys of earlier kernels is not reused, and trials are whole groups of eight
steps (the library's launches of four steps)."""
import json

import torch

from paper_1507_02509_amd import _lib as L
from paper_1507_02509_amd import autotune


class Stub:
    """A lattice, and an ensemble of itself, that records what is asked of it."""
    device, form, nx, ny, steps, ctx = "cpu", L.F32DEV_F32, 512, 512, 0, None

    def __init__(self):
        self.params = L.Params()
        self.calls, self.set = [], []
        self.buf = torch.zeros(4)
        self.members = [self]
        self.lib = self

    def lbm_set_step(self, ctx, n):
        return 0

    def state_buffer(self):
        return self.buf

    def set_fusion(self, *a):
        self.set.append(("fusion", *a))

    def set_tile(self, *a):
        self.set.append(("tile", *a))

    def step(self, n, persistent=False):
        self.calls.append(n)


def test_keys_and_trials(monkeypatch, tmp_path):
    path = tmp_path / "autotune.json"
    monkeypatch.setenv("KBC_AUTOTUNE_CACHE", str(path))
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda d: "gpu")
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    s = Stub()
    monkeypatch.setattr(autotune, "_time", lambda run, steps, reps: run(steps) or float(len(s.calls)))
    new = autotune._sim_key(s), autotune._ens_key(s) + "|per-step"
    old = [k.replace("sim4|", "sim3|").replace("ensemble4|", "ensemble3|") for k in new]
    assert set(old).isdisjoint(new)
    path.write_text(json.dumps({k: {"tile": ["fused", 24, False]} for k in old}))
    for tune in (autotune.tune_sim, autotune.tune_ensemble):
        for kw in ({}, {"steps": 4}, {"steps": 9}):
            s.calls.clear()
            best, timings = tune(s, use_cache=False, **kw)
            assert s.calls and all(n % 8 == 0 for n in s.calls), (tune, kw, s.calls)
        s.calls.clear()
        best, timings = tune(s)
        assert s.calls and best == next(iter(timings)), "a choice made for earlier kernels was reused"
        s.calls.clear()
        assert tune(s)[0] == best and not s.calls      # its own choice is
