"""Keys of cached launch shapes (host)."""
from types import SimpleNamespace

from paper_2506_07430_amd import autotune


def test_shapes_of_another_meaning_are_not_applied(monkeypatch, tmp_path):
    """A cache written when `groups` counted list-entry groups holds nothing for networks whose
    items are now segments of parents, nor does one of a later meaning."""
    monkeypatch.setattr(autotune, "_device_name", lambda: "gfx950:256cu")
    ham, ans = SimpleNamespace(n=24, na=12, nb=12), SimpleNamespace(widths=(128, 128), precision=1)
    key = autotune.problem_key(ham, ans, 4096)
    path = str(tmp_path / "cache.json")
    autotune.store_cache("gfx950:256cu|n24|a12b12|w128x128|p1|B4096", {"shape": {"groups": 8}}, path)
    assert key not in autotune.load_cache(path)
    autotune.store_cache(key, {"shape": {"groups": 4}}, path)
    assert autotune.load_cache(path)[key] == {"shape": {"groups": 4}}
    monkeypatch.setattr(autotune, "SHAPE_VERSION", autotune.SHAPE_VERSION + 1)
    assert autotune.problem_key(ham, ans, 4096) not in autotune.load_cache(path)
