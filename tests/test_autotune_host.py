"""The autotuner's choice of what to time, with a solver that only counts."""
import json
import types

import pytest

from paper_1206_3229_amd import autotune
from paper_1206_3229_amd import inputs as I
from paper_1206_3229_amd import vlasov as V

ARCH = "gfx950"


class _Event:
    def __init__(self, enable_timing):
        pass

    def record(self):
        pass

    def elapsed_time(self, other):
        return 1.0


@pytest.fixture
def timed(monkeypatch, tmp_path):
    """Launch shapes that tune() sets, in turn; no GPU."""
    import torch
    shapes = []
    solver = types.SimpleNamespace(set_tuning=lambda *s: shapes.append(s), step=lambda n: None, close=lambda: None)
    monkeypatch.setattr(autotune, "V", types.SimpleNamespace(Solver=lambda p, f0: solver,
                                                             tuning_candidates=V.tuning_candidates))
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: types.SimpleNamespace(gcnArchName=ARCH))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "Event", _Event)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setenv("VLASOV_TUNE_CACHE", str(tmp_path / "tune.json"))
    return shapes


def test_shapes_of_the_same_kernels_are_timed_once(timed):
    p, f0, _ = I.hmf_waterbag_small()
    best = autotune.tune(p, f0)
    assert len({s[1:] for s in timed}) == len(timed) == len({c[1:] for c in V.tuning_candidates()})
    assert len(best["table"]) == len(V.tuning_candidates())


def test_times_of_earlier_kernels_are_not_taken_from_the_cache(timed, tmp_path):
    p, f0, _ = I.hmf_waterbag_small()
    old = f"{ARCH}|s{p.storage}|{p.nx}x{p.np_}|bc{p.bc_x}{p.bc_p}|dt{p.dt!r}|v3"
    (tmp_path / "tune.json").write_text(json.dumps({old: {"us_per_step": 0.0}}))
    assert autotune.tune(p, f0)["us_per_step"] > 0.0 and timed
    del timed[:]
    assert autotune.tune(p, f0)["us_per_step"] > 0.0 and not timed  # its own entry is
