"""The tuner's cache file: a pick is kept for the library it was measured with."""
import json
import types

import pytest
import torch

from paper_1902_05942_amd import autotune


@pytest.fixture
def tuner(monkeypatch, tmp_path):
    monkeypatch.setenv("PF_AUTOTUNE_CACHE", str(tmp_path / "picks.json"))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: types.SimpleNamespace(name="gpu", multi_processor_count=256))
    frames = [{"px": torch.zeros(1000)}]
    calls = []

    def tune(best):
        def time_config(mvf, f, block, agg, reps=5):
            calls.append((block, agg))
            return 1.0 if (block, agg) == best else 2.0

        monkeypatch.setattr(autotune, "time_config", time_config)
        del calls[:]
        return autotune.tune(None, frames)[:2], len(calls)

    return tune


def test_a_pick_is_reused(tuner):
    assert tuner((1024, 4096)) == ((1024, 4096), 25)
    assert tuner((512, 4096)) == ((1024, 4096), 0)


def test_another_library_is_measured_again(tuner, monkeypatch, tmp_path):
    other = tmp_path / "libpf.so"
    other.write_bytes(b"another build")
    assert tuner((1024, 4096)) == ((1024, 4096), 25)
    if hasattr(autotune, "library_digest"):
        autotune.library_digest.cache_clear()
    monkeypatch.setattr(autotune, "LIB_PATH", str(other), raising=False)
    try:
        assert tuner((512, 4096)) == ((512, 4096), 25)
    finally:
        if hasattr(autotune, "library_digest"):
            autotune.library_digest.cache_clear()


def test_a_file_of_before_is_kept(tuner, tmp_path):
    path = tmp_path / "picks.json"
    old = {"gpu|256|1000": {"block": 64, "agg": 64, "ms": {"64/64": 1.0}}}
    path.write_text(json.dumps(old))
    assert tuner((512, 4096)) == ((512, 4096), 25)
    kept = json.loads(path.read_text())
    assert kept["gpu|256|1000"] == old["gpu|256|1000"] and len(kept) == 2
