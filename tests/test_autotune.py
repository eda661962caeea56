"""The autotuner's saved configurations and what it times: a configuration
saved for another build of the library is not applied, and a step without a
head pass is not tuned."""
import hashlib
import json
import types

import pytest
import torch

import rt_inputs as ri
from paper_1304_7126_amd import autotune


class StubBatch:
    """A batch whose configuration can be set and timed without a GPU."""
    fp32 = True
    boxes = [types.SimpleNamespace(n=(16, 16, 16), M=1), types.SimpleNamespace(n=(24, 24, 24), M=3)]

    def __init__(self):
        self.config = None

    def set_tuning(self, *config):
        self.config = config

    def snapshot(self):
        return None

    def restore(self, snap):
        pass

    def step(self, dt, n):
        pass

    def synchronize(self):
        pass


@pytest.fixture
def tune(tmp_path, monkeypatch):
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "tune.json"))
    monkeypatch.setattr(autotune, "_gpu_name", lambda: "some GPU")

    def use_library(content):
        lib = tmp_path / hashlib.sha1(content).hexdigest()
        lib.write_bytes(content)
        monkeypatch.setattr(autotune, "LIB_PATH", str(lib), raising=False)

    use_library(b"a build")
    return use_library


def test_saved_configuration_belongs_to_one_build(tune):
    b = StubBatch()
    first = autotune.tune_batch(b, 1.0, trial_steps=1)
    assert not first["cached"]
    assert autotune.tune_batch(b, 1.0)["cached"] and b.config == (*first["config"], 1)
    tune(b"another build")
    assert not autotune.tune_batch(b, 1.0, trial_steps=1)["cached"]
    tune(b"a build")
    assert autotune.tune_batch(b, 1.0)["cached"]


def test_configuration_saved_without_a_build_is_not_applied(tune):
    b = StubBatch()
    shapes = sorted((x.n, x.M) for x in b.boxes)
    key = "batch:" + hashlib.sha1(json.dumps([shapes, True, "some GPU"]).encode()).hexdigest()[:16]
    with open(autotune.CACHE, "w") as f:
        json.dump({key: {"config": [64, 1, 65536], "ms_per_step": 1.0}}, f)
    r = autotune.tune_batch(b, 1.0, trial_steps=1)
    assert not r["cached"] and r["config"] != [64, 1, 65536]


@pytest.mark.gpu
@pytest.mark.parametrize("transport,chem,trials", [("auto", "auto", 0), ("zmarch", "one-pass", 0), ("cell", "auto", 5),
                                                   ("auto", "two-pass", 5)])
def test_tune_grid_times_only_a_step_that_has_a_head_pass(transport, chem, trials):
    from paper_1304_7126_amd import RTContext
    w = ri.lognormal_box(12, 6.6 * 12 / 128, 2, steps=2, seed=3)
    c = RTContext.for_workload(w, fp32=True)
    c.load_state(ri.initial_state(w))
    c.set_transport_path(transport)
    c.set_chem_path(chem)
    x, cur = c.xHII.clone(), c.current
    r = autotune.tune_grid(c, c.courant_dt())
    assert len(r["trials"]) == trials and (r["head_attempts"] > 0) == (trials > 0)
    c.set_tuning(r["head_attempts"])
    assert torch.equal(c.xHII, x) and c.current == cur
