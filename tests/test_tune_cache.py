"""The autotuner's cache on disk, with the device calls replaced: an entry
measured on kernels of another revision is measured again, others are applied."""
import json
import types

import torch


def test_entries_of_other_kernels_are_measured_again(tmp_path, monkeypatch):
    from paper_2505_22631_amd import tune
    path = tmp_path / "cache.json"
    monkeypatch.setenv("OIM_TUNE_CACHE", str(path))
    monkeypatch.setattr(tune, "bucket", lambda problem, R, q: f"R{R}|q{q}")
    applied, measured = [], []
    monkeypatch.setattr(tune, "oim_set_tuning", lambda h, q, *shape: applied.append(shape))

    def autotune(*args, **kw):
        measured.append(kw["trial_steps"])
        return {"block": 512, "slices_per_wave": 1, "rows_per_lane": 2, "ms": 1.0, "tried": []}

    monkeypatch.setattr(tune, "oim_autotune", autotune)
    old = {"block": 1024, "slices_per_wave": 2, "rows_per_lane": 1, "trial_ms": 3.0, "trial_steps": 5,
           "tried": []}
    other = dict(old, kernels=tune.KERNELS)
    path.write_text(json.dumps({"R2|q2": old, "R2|q3": other, "R2|q5": dict(old, kernels=-1)}))
    prob = types.SimpleNamespace(handle=1, n=4)
    K = torch.zeros(5)
    call = lambda q: tune.tuned(prob, torch.zeros(2, 4), K, K, K, None, q=q, dt=0.1)  # noqa: E731

    e, now = call(2)  # no revision: measured, stored, then applied
    assert now and e["block"] == 512 and measured == [5] and not applied
    e, now = call(2)
    assert not now and applied == [(512, 1, 2)]
    e, now = call(3)  # this revision: applied
    assert not now and applied[-1] == (1024, 2, 1) and measured == [5]
    assert call(5)[1] and measured == [5, 5]  # another one
    stored = json.loads(path.read_text())
    assert stored["R2|q2"]["kernels"] == stored["R2|q5"]["kernels"] == tune.KERNELS
    assert stored["R2|q3"] == other
