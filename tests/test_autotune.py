"""The launch-shape tuner's choice and its cache, without a device: which of some
timed shapes is taken, and that shapes stored for other kernels are not."""
import json

import pytest
import torch

from paper_2605_03208_amd import autotune, kc


class _Ctx:
    """Stands in for a context: every shape has a time of its own."""

    def __init__(self, ms):
        self.ms, self.shape, self.timing = ms, None, False

    def enable_timing(self, on=True):
        self.timing = on

    def set_tuning(self, op, **cand):
        self.shape = cand

    def kernel_ms(self, op):
        return self.ms[self.shape["grid_per_cu"]]


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("KC_TUNE_CACHE", str(path))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    return path


@pytest.mark.parametrize("ms,best", [({0: 1.004, 4: 1.0, 8: 1.3}, 0), ({0: 1.006, 4: 1.0, 8: 1.3}, 4),
                                     ({0: 1.0, 4: 1.1, 8: 1.2}, 0), ({2: 1.0, 4: 1.004}, 2)])
def test_the_rule_is_taken_within_its_margin(cache, ms, best):
    ctx = _Ctx(ms)
    cands = [dict(grid_per_cu=g) for g in ms]
    r = autotune.tune(ctx, kc.OP_RESTORE, lambda: None, signature="t", candidates=cands)
    assert r["best"] == dict(grid_per_cu=best) == ctx.shape and not r["cached"]
    assert autotune.tune(ctx, kc.OP_RESTORE, lambda: None, signature="t", candidates=cands)["cached"]


def test_shapes_of_other_kernels_are_not_used(cache, monkeypatch):
    hip = getattr(torch.version, "hip", None) or "unknown"
    old = [f"{autotune.ARCH}|{hip}|snapshot|t", f"{autotune.ARCH}|{hip}|kernels{autotune.KERNELS - 1}|snapshot|t"]
    cache.write_text(json.dumps({k: dict(best=dict(grid_per_cu=4), table=[]) for k in old}))
    key = autotune.cache_key(kc.OP_SNAPSHOT, "t")
    assert key not in old and autotune.lookup(key) is None
    r = autotune.tune(_Ctx({0: 1.0, 4: 1.2}), kc.OP_SNAPSHOT, lambda: None, signature="t",
                      candidates=[dict(grid_per_cu=0), dict(grid_per_cu=4)])
    assert r["best"] == dict(grid_per_cu=0) and not r["cached"]


def test_shipped_shapes_are_what_the_tuner_picks():
    with open(autotune.SHIPPED) as f:
        shipped = json.load(f)
    assert shipped
    for key, entry in shipped.items():
        assert f"|kernels{autotune.KERNELS}|" in key
        assert entry["best"] == autotune.pick(entry["table"]), key
