"""The Python extension beside the library: the library's build does not depend on it, and it serves the torch and the interpreter it was
built with alone."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2503_01066_amd import build as B


@pytest.fixture
def only_marshal(monkeypatch, tmp_path):
    """A build that finds everything but the extension up to date, in a folder of its own."""
    target = tmp_path / os.path.basename(B.MARSHAL)
    target.write_bytes(b"of older sources")
    monkeypatch.setattr(B, "MARSHAL", str(target))
    monkeypatch.setattr(B, "_marshal_stamp", lambda: str(tmp_path / "stamp"))
    monkeypatch.setattr(B, "_stale", lambda t, deps: t == str(target) and target.read_bytes()[:4] != b"\x7fELF")
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
    assert not B._marshal_stale()


def test_extension_is_built_again_for_another_torch(monkeypatch, only_marshal):
    B.build(verbose=False)
    monkeypatch.setattr(B, "torch_build", lambda: "another torch")
    assert B._marshal_stale()


@pytest.mark.parametrize("change,used", [("pass", True), ("torch.__version__ = '2.10.1'", False), ("torch.version.git_version = 'f00'", False)])
def test_extension_is_used_with_its_own_torch_alone(change, used):
    assert B.MARSHAL.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and os.path.exists(B.MARSHAL)
    code = "import torch; %s; from paper_2503_01066_amd import binding; print(binding._marshal is not None)" % change
    out = subprocess.run([sys.executable, "-c", code], cwd=B.ROOT, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.split() == [str(used)], (out.stdout, out.stderr)
