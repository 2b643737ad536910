"""Tuning records written by an earlier version of the library (no GPU)."""
import types

import torch

from paper_1708_04710_amd import _binding, api, autotune


def test_records_of_earlier_versions_are_searched_anew(monkeypatch):
    """A setting other than the built-in one turns the blocks solved apart off;
    version 0.2 had none, so what was the fastest for it (the 400-point torus to
    dimension 3: 12 ms) is not what is now (4.3)."""
    f = types.SimpleNamespace(view=types.SimpleNamespace(m=1000, nnz=3000), device="cuda:0")
    applied = []
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: types.SimpleNamespace(gcnArchName="gfx950"))
    monkeypatch.setattr(api, "set_tuning", lambda t, device=None: applied.append(dict(t)))
    monkeypatch.setattr(api, "time_candidates", lambda f, cands, **kw: ([1.0] * len(cands), 0, None))
    old = {**api.default_tuning(), "lane_steps_few": 8}
    cache = autotune.TuneCache()
    cache.put(autotune.cache_key("gfx950", "pms-gfx950 0.2", 1000, 3000), dict(tuning=old, graph_rounds=0, ms=12.0, scored=3))
    rec = autotune.autotune(f, cache=cache, grid={"lane_steps_few": (0, 8)})
    assert not rec["cached"] and rec["tuning"] == api.default_tuning() and applied[-1] == api.default_tuning()
    again = autotune.autotune(f, cache=cache, grid={"lane_steps_few": (0, 8)})
    assert again["cached"] and again["key"].split("/")[1] == _binding.load().pms_version().decode()
