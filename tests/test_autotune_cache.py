"""The autotuner's cache file: a choice is reused only for the kernels it was timed on
(the library's calls replaced by stand-ins; no GPU)."""
import json
import types

import torch

from paper_2311_13081_amd import sim as sim_mod


class Handle(sim_mod.QuadSim):
    def __init__(self):  # no device
        self.N, self.cfg, self.device, self.h = 256, {"flags": 7}, torch.device("cuda", 0), None
        self.set, self.timed = [], 0

        def sim_autotune(h, actor, T, stream, v, ms):
            self.timed += 1
            v._obj.value, ms._obj.value = 5, 0.25
            return 0

        self.L = types.SimpleNamespace(sim_autotune=sim_autotune)

    def set_variant(self, variant, spl=0, graph=True):
        self.set.append((variant, spl))

    def get_variant(self):
        return 5, 100, 1


def test_entries_of_other_kernels_are_not_used(tmp_path, monkeypatch):
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: types.SimpleNamespace(gcnArchName="gfx950:sramecc+"))
    monkeypatch.setattr(sim_mod, "_ptr", lambda t: t)
    monkeypatch.setattr(sim_mod, "_stream", lambda: None)
    path = tmp_path / "tune.json"
    old = {"N=256 flags=7 T=100 arch=gfx950": {"variant": 3, "steps_per_launch": 0, "ms": 0.5}}
    path.write_text(json.dumps(old))
    a = Handle()
    assert a.autotune("actor", 100, cache=str(path)) == (5, 0.25)
    assert a.timed == 1 and a.set == []          # timed again, the old choice not set
    table = json.loads(path.read_text())
    assert set(old) < set(table) and len(table) == 2  # the old entry stays for its build
    b = Handle()
    assert b.autotune("actor", 100, cache=str(path)) == (5, 0.25)
    assert b.timed == 0 and b.set == [(5, 100)]  # the new one is reused
    monkeypatch.setattr(sim_mod, "VARIANT_KERNELS", sim_mod.VARIANT_KERNELS + 1)
    c = Handle()
    c.autotune("actor", 100, cache=str(path))
    assert c.timed == 1
