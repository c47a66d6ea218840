"""The tuner times each configuration once (on a stand-in for the solver)."""
import torch

from paper_2103_05694_amd import autotune


def test_no_two_candidates_differ_in_an_option_without_effect(monkeypatch):
    seen = []

    def solve(field, h, sources, **kw):
        out = kw.pop("out", None)
        kw.pop("packed", None)
        kw.pop("check_status", None)
        seen.append(tuple(sorted((k, str(v)) for k, v in kw.items())))
        return out.zero_() if out is not None else torch.zeros_like(field)

    monkeypatch.setattr(autotune.api, "solve", solve)
    monkeypatch.setattr(autotune.api, "status", lambda *a, **k: None)
    monkeypatch.setattr(autotune, "_time", lambda fn, reps: 1.0 + 0.0 * len(seen))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    e = autotune.tune(torch.ones(8, 8, dtype=torch.float64), 1.0, torch.tensor([0]), save=False, log=lambda *a: None)
    keys = [tuple(sorted((k, str(v)) for k, v in c.items() if k not in ("packed", "ms"))) for c in e["candidates"]]
    assert len(keys) == len(set(keys)) > 50
    assert e["packed"] is False
