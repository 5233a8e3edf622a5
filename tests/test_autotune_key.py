"""The autotuner's cache on disk: a shape is taken over only from the library
that it was timed with."""
import json
import types

import pytest


@pytest.fixture
def tuner(tmp_path, monkeypatch):
    from paper_2506_02741_amd import _lib, autotune
    path = tmp_path / "autotune.json"
    monkeypatch.setenv("VTGS_AUTOTUNE_CACHE", str(path))
    timed = []

    def fake(keyframes, views, mode, tile, batch, reps):
        timed.append((tile, batch))
        return 1.0 + abs(tile - 8) + abs(batch - 512) / 100, 1
    monkeypatch.setattr(autotune, "_time_config", fake)
    monkeypatch.setattr(autotune, "_arch", lambda: "gfx950")
    kf = types.SimpleNamespace(n=1000)
    view = types.SimpleNamespace(cam=types.SimpleNamespace(width=64, height=48), kf_first=0, kf_count=1)

    def library(data):
        (tmp_path / "lib.so").write_bytes(data)
        monkeypatch.setattr(_lib, "LIB_PATH", str(tmp_path / "lib.so"))
        getattr(_lib, "revision", types.SimpleNamespace(cache_clear=lambda: None)).cache_clear()

    def tune():
        timed.clear()
        prm, _ = autotune.tune([kf], [view])
        return (prm.tile, prm.batch), len(timed)
    yield types.SimpleNamespace(library=library, tune=tune, path=path)
    getattr(_lib, "revision", types.SimpleNamespace(cache_clear=lambda: None)).cache_clear()


def test_shapes_of_another_library_are_timed_again(tuner):
    from paper_2506_02741_amd import _lib
    _lib.load()  # (the real one, before its path is replaced)
    tuner.library(b"one")
    assert tuner.tune() == ((8, 512), 9)
    assert tuner.tune() == ((8, 512), 0)  # kept
    cache = json.loads(tuner.path.read_text())
    for e in cache.values():              # another winner, as other kernels may have
        e.update(tile=32, batch=128)
    tuner.path.write_text(json.dumps(cache))
    assert tuner.tune() == ((32, 128), 0)
    tuner.library(b"two")
    assert tuner.tune() == ((8, 512), 9)


def test_shapes_kept_without_a_library_are_not_taken_over(tuner):
    from paper_2506_02741_amd import _lib
    _lib.load()
    tuner.library(b"one")
    tuner.path.write_text(json.dumps({"gfx950|track|v1|64x48|g1024": dict(tile=32, batch=128)}))
    assert tuner.tune() == ((8, 512), 9)
