"""The schedule tuner's cache on disk (no GPU): a schedule timed with another
build of the library, whose launches it may no longer describe, is not taken."""
import json

from paper_1706_01094_amd import autotune
from paper_1706_01094_amd import mclg as M

SHAPE = dict(L=1 << 20, rho=50.0, u0=0.1, C=10, lam=(1, 1), n_max=255, device_name="card")


def test_the_signature_names_the_build(tmp_path, monkeypatch):
    here = autotune.signature(**SHAPE)
    assert here == autotune.signature(**SHAPE) != autotune.signature(**dict(SHAPE, C=5))
    other = tmp_path / "lib.so"
    for content in (b"another build", b"and another"):
        other.write_bytes(content)
        monkeypatch.setattr(M, "LIB_PATH", str(other))
        assert autotune.signature(**SHAPE) != here
        here = autotune.signature(**SHAPE)


def test_an_older_entry_is_not_taken(tmp_path, monkeypatch):
    """With the cache of another build, tune() goes on to time a lattice."""
    import torch
    cache = tmp_path / "cache.json"
    other = tmp_path / "lib.so"
    other.write_bytes(b"another build")
    with monkeypatch.context() as m:
        m.setattr(M, "LIB_PATH", str(other))
        old = autotune.signature(1 << 20, 50.0, 0.1, 10, (1, 1), 255, "card")
    cache.write_text(json.dumps({old: {"schedule": [1, 768, 4096], "seconds_per_step": 1.0, "trials": []}}))
    monkeypatch.setattr(autotune, "CACHE_PATH", str(cache))
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda i: "card")

    class Timed(Exception):
        pass

    def lattice(*a, **k):
        raise Timed

    monkeypatch.setattr(M, "Lattice", lattice)
    try:
        autotune.tune(1 << 20, 50.0, 0.1)
        raise AssertionError("the schedule of another build was taken")
    except Timed:
        pass
