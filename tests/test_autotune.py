"""What the autotuner keeps, with the timings given: no device needed."""
import json
from types import SimpleNamespace

import pytest

import paper_2608_18065_amd as pm
from paper_2608_18065_amd import autotune


class FakeModel:
    def __init__(self, dtype=pm.F32):
        self.desc = SimpleNamespace(dim=1, hidden=64, complex_head=0, compute_dtype=dtype)
        self.N, self.device, self.tunables = 16, 0, {}

    def set_tunable(self, key, value):
        self.tunables[key] = value


@pytest.fixture
def timed(monkeypatch):
    """(sampling, evaluation) ms by sample_r; other phases the same for every value"""
    ms = {}
    monkeypatch.setattr(autotune.torch.cuda, "get_device_properties",
                        lambda d: SimpleNamespace(gcnArchName="gfx950:x"))
    monkeypatch.setattr(autotune, "_time_phase", lambda m, ham, Ns, form, phases, reps:
                        ms[m.tunables["sample_r"]][0] if phases == ("sample",) else 1.0)
    monkeypatch.setattr(autotune, "_time_evaluation", lambda m, Ns, reps:
                        ms[m.tunables["sample_r"]][1], raising=False)
    return ms


@pytest.mark.parametrize("ms,best", [
    ({0: (1.00, 1.0), 1: (0.99, 1.0), 4: (0.98, 1.0)}, 0),     # the same kernels, timing noise
    ({0: (1.0, 0.1), 1: (0.9, 0.6), 4: (0.9, 0.6)}, 0),        # faster sampling, slower evaluation
    ({0: (1.0, 1.0), 1: (1.2, 1.0), 4: (0.7, 0.8)}, 4),        # faster in both
])
def test_sample_r_leaves_the_matrix_cores_only_for_a_gain(timed, tmp_path, ms, best):
    timed.update(ms)
    m = FakeModel()
    cache = str(tmp_path / "t.json")
    res = autotune.tune(m, None, 256, cache=cache)
    assert res["sample_r"][0] == best and m.tunables["sample_r"] == best
    assert res["sample_r"][1][best] == min(res["sample_r"][1].values())
    fresh = FakeModel()
    assert autotune.apply(fresh, 256, cache=cache)["sample_r"] == best
    assert autotune.apply(FakeModel(pm.F64), 256, cache=cache) == {}


def test_entries_of_before_the_matrix_core_recurrence(timed, tmp_path):
    # their sample_r was the built-in choice's form of the time, 1 or 4
    cache = tmp_path / "t.json"
    entry = {"gram_split": 4, "eloc_grid": 512, "sample_r": 1, "jac_parts": 2}
    cache.write_text(json.dumps({"gfx950/dim1/H64/N16/Ns256/cplx0/form%d" % f: entry
                                 for f in (pm.FORM_FP64_REF, pm.FORM_BF16_FP64)}))
    m = FakeModel()
    assert autotune.apply(m, 256, cache=str(cache)) == {"gram_split": 4, "eloc_grid": 512}
    assert m.tunables == {"gram_split": 4, "eloc_grid": 512}
    assert autotune.apply(m, 256, form=pm.FORM_FP64_REF, cache=str(cache)) == {"eloc_grid": 512}
    assert autotune.apply(m, 512, cache=str(cache)) == {}
