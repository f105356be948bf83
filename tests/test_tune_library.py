"""The autotune cache belongs to one build of the library (no device)."""
from paper_2012_04838_amd import psdns, tune
from tests.test_tune_cache import FakePlan


def _library(tmp_path, monkeypatch, name, content):
    path = tmp_path / name
    path.write_bytes(content)
    monkeypatch.setattr(psdns, "LIB_PATH", str(path))


def test_key_follows_the_kernels_and_not_only_their_descriptions(tmp_path, monkeypatch):
    keys = []
    # two builds whose schedule descriptions agree, and the first again under another name
    for name, content in (("a.so", b"separate passes"), ("b.so", b"plane pass"), ("c.so", b"separate passes")):
        _library(tmp_path, monkeypatch, name, content)
        keys.append(tune.cache_key("dev", FakePlan()))
    assert keys[0] != keys[1]
    assert keys[0] == keys[2]


def test_a_rebuilt_library_is_timed_again(tmp_path, monkeypatch):
    cache = str(tmp_path / "tune.json")
    for name, content, timed in (("a.so", b"old", 1), ("b.so", b"new", 1), ("c.so", b"old", 0)):
        _library(tmp_path, monkeypatch, name, content)
        p = FakePlan()
        assert tune.autotune(p, None, None, cache=tune.TuneCache(cache), device="dev") == 2
        assert p.timed == timed
