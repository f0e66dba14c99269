"""The autotuner's cache key: another build of the library, layout, periodic axis
or kind of segment is another entry."""
from types import SimpleNamespace

from paper_1307_4703_amd import tune


def _lat(**kw):
    d = dict(nx=64, ny=32, storage="f32", layout="paired", periodic=(False, False), segments={},
             info=lambda: {"n_fluid": 1000})
    return SimpleNamespace(**(d | kw))


def test_keys_tell_forms_apart(monkeypatch, tmp_path):
    keys = [tune._key([_lat(**kw)], "lattice2")
            for kw in ({}, {"layout": "planes"}, {"periodic": (True, False)}, {"storage": "f16"},
                       {"segments": {2: ("pressure", (0, 1), 1.0, 0.0, False)}})]
    keys.append(tune._key([_lat()], "cde4"))
    assert len(set(keys)) == len(keys)
    assert tune._key([_lat()], "lattice2") == keys[0]
    # another build of the library
    lib = tmp_path / "libgg.so"
    lib.write_bytes(b"one")
    one = tune._library(str(lib))
    other = tmp_path / "other.so"
    other.write_bytes(b"two")
    assert tune._library(str(other)) != one
    monkeypatch.setattr(tune, "_library", lambda: one)
    assert tune._key([_lat()], "lattice2") != keys[0]
