"""The Python extension beside the library: the library's build does not depend on it."""
import os

import pytest

from paper_2503_01066_amd import build as B


@pytest.fixture
def only_marshal(monkeypatch, tmp_path):
    """A build that finds everything but the extension up to date, in a folder of its own."""
    target = tmp_path / os.path.basename(B.MARSHAL)
    target.write_bytes(b"of older sources")
    monkeypatch.setattr(B, "MARSHAL", str(target))
    monkeypatch.setattr(B, "_stale", lambda t, deps: t == str(target))
    return target


@pytest.mark.parametrize("compiler", ["false", "no such compiler"])
def test_library_is_built_where_the_extension_cannot_be(monkeypatch, only_marshal, capfd, compiler):
    monkeypatch.setenv("CXX", compiler)
    assert B.build(verbose=False) == B.LIB
    assert not only_marshal.exists()
    assert compiler in capfd.readouterr().err


def test_extension_is_built(only_marshal):
    B.build(verbose=False)
    assert only_marshal.read_bytes()[:4] == b"\x7fELF"
