"""The build and what it leaves (CPU only): the library does not depend on the binding's compiled module, and
a module of another torch is not used."""
import os
import subprocess
import sys
import types

import pytest

import paper_2305_08872_amd as am
from paper_2305_08872_amd import binding
from paper_2305_08872_amd import build as hip_build


@pytest.mark.parametrize("step", ["_compile_marshal", "_link_marshal"])
def test_the_library_is_built_without_the_compiled_module(monkeypatch, tmp_path, capsys, step):
    """No g++, no Python or torch headers: the library all the same, no module (nor an old one)."""
    if not os.path.exists(am.library_path()):
        hip_build.build()
    objects = {s: os.path.join(hip_build.OBJ_DIR, os.path.splitext(s)[0] + ".o") for s in hip_build.SOURCES}
    if not all(os.path.exists(o) for o in objects.values()):
        hip_build.build()

    def missing(*_):
        raise FileNotFoundError("g++")

    monkeypatch.setattr(hip_build, "_compile", lambda src: objects[src])
    monkeypatch.setattr(hip_build, "LIB_PATH", str(tmp_path / "libamulet.so"))
    monkeypatch.setattr(hip_build, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(hip_build, "_compile_marshal", lambda: "")
    monkeypatch.setattr(hip_build, step, missing)
    (tmp_path / "_marshal.so").write_bytes(b"an old one")
    assert hip_build.build() == str(tmp_path / "libamulet.so")
    assert os.listdir(tmp_path) == ["libamulet.so"]
    assert "not built" in capsys.readouterr().err


def test_a_module_of_another_torch_or_without_a_stamp_is_not_used(monkeypatch):
    name = binding.__package__ + "._marshal"
    for stamp, used in ((hip_build.torch_build(), True), ("2.0.0 0123abcd", False), (None, False)):
        module = types.SimpleNamespace() if stamp is None else types.SimpleNamespace(built_for_torch=stamp)
        monkeypatch.setitem(sys.modules, name, module)
        assert (binding._compiled_marshalling() is module) is used
    monkeypatch.setitem(sys.modules, name, None)      # not there: import raises
    assert binding._compiled_marshalling() is None


def test_the_module_built_here_carries_this_torch_and_python():
    if not os.path.exists(hip_build.MARSHAL_PATH):
        hip_build.build()
    out = subprocess.check_output(
        [sys.executable, "-c", "import torch, paper_2305_08872_amd as am; am.load_library(); "
         "from paper_2305_08872_amd import binding; print(binding._marshal.__file__)"],
        text=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(hip_build.__file__))))
    assert out.strip().endswith(os.path.basename(hip_build.MARSHAL_PATH)) and "cpython" in out
