"""The autotuner's JSON cache across library builds, with the library's calls
replaced by counters: a choice timed with another build (or before builds were
noted) is not applied but timed again and replaced; one of this build is applied
without timing."""
import json
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2510_12053_amd import autotune
import paper_2510_12053_amd.ccgpu as cg


@pytest.fixture
def calls(monkeypatch, tmp_path):
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"one build")
    seen = dict(steps=0, dense=[])
    monkeypatch.setattr(cg, "LIB_PATH", str(lib))
    monkeypatch.setattr(cg, "cc_batch_tuning", lambda *a: None)
    monkeypatch.setattr(cg, "cc_dense_tuning", lambda ctx, rows, chunk: seen["dense"].append(rows))

    def step(*a, **k):
        seen["steps"] += 1
    monkeypatch.setattr(cg, "cc_step_batch", step)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    return seen, lib, str(tmp_path / "tune" / "cache.json")


def _tune(path):
    par = types.SimpleNamespace(precision=cg.FP32_MIXED, sweep=cg.SWEEP_JACOBI)
    x = [torch.zeros(4, 3)]
    return autotune.tune(None, [0], x, x, [None, None], 1.0 / 60, par, 1e-6, None, 1000, True, False,
                         cache_path=path, device_arch="gfx950")


def test_choice_of_another_build_is_timed_again(calls):
    seen, lib, path = calls
    first, table = _tune(path)
    assert table and seen["steps"] > 0
    steps = seen["steps"]
    assert _tune(path) == (first, None)
    assert seen["steps"] == steps
    lib.write_bytes(b"another build")
    assert _tune(path)[1] is not None and seen["steps"] > steps
    steps = seen["steps"]
    assert _tune(path)[1] is None and seen["steps"] == steps


def test_entry_without_a_build_is_not_applied(calls):
    seen, lib, path = calls
    key = autotune.cache_key("gfx950", 1, 0, True, 1000, 1)
    autotune._save(path, {key: {"lanes": 16, "iters_per_graph": 1, "dense_rows": 2}, "other": {"lanes": 16}})
    assert _tune(path)[1] is not None
    table = json.load(open(path))
    assert "build" in table[key] and table["other"] == {"lanes": 16}
