"""The cache keeps a choice that leaves a size to the library's own form."""
from paper_1210_7774_amd import tunecache as T


def test_library_form_roundtrip(tmp_path):
    p = str(tmp_path / "tune.json")
    k = T.key("dev", "f64|rbgs|nu2,2", "poisson2d", [1023])
    c = {1023: (32, None), 511: (32, True), 255: (8, False)}
    T.store(p, k, c)
    assert T.load(p, k) == c
    # an entry written when false stood for the library's form as well is not read
    assert not k.startswith("v1|")
