"""The binding's native module: it is loaded only if it was built from the present sources for the present Python and torch,
and the library loads without it."""
import os
import subprocess

import pytest
import torch

from paper_1804_08066_amd import build, mqgrad


def test_the_module_is_named_by_what_it_was_built_from(monkeypatch, tmp_path):
    here = build.marshal_path()
    assert build.marshal_path() == here
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".other")
    other_torch = build.marshal_path()
    monkeypatch.undo()
    source = tmp_path / build.MARSHAL_SOURCE
    with open(os.path.join(build.CSRC, build.MARSHAL_SOURCE)) as f:
        source.write_text(f.read() + "\n")
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    assert len({here, other_torch, build.marshal_path()}) == 3


def test_a_module_of_another_torch_is_not_current(monkeypatch):
    if not os.path.exists(build.marshal_path()):
        build._build_marshal(False)
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".other")
    assert build.needs_build()


@pytest.mark.parametrize("compiler", ["/nonexistent/c++", "/bin/false"])
def test_the_binding_makes_its_own_tables_where_the_module_cannot_be_built(monkeypatch, tmp_path, compiler):
    monkeypatch.setattr(build, "marshal_path", lambda: str(tmp_path / "_marshal.so"))
    monkeypatch.setenv("CXX", compiler)
    with pytest.warns(UserWarning, match="argument tables"):
        assert build.load_marshal() is None
    assert mqgrad._NoTables.pointers([], [], 0, 4, 512, 0) is None


def test_a_file_that_is_no_module_is_passed_over(monkeypatch, tmp_path):
    path = tmp_path / "_marshal.so"
    path.write_bytes(b"not a library")
    monkeypatch.setattr(build, "marshal_path", lambda: str(path))
    with pytest.warns(UserWarning, match="argument tables"):
        assert build.load_marshal() is None


def test_the_library_loads_without_the_module(tmp_path):
    code = ("import warnings; warnings.simplefilter('ignore')\n"
            "from paper_1804_08066_amd import build, mqgrad\n"
            "build.marshal_path = lambda: %r\n"
            "assert mqgrad.mqg_packed_words(33, 4) == 5 and mqgrad._marshal is mqgrad._NoTables" % str(tmp_path / "none.so"))
    root = os.path.dirname(os.path.dirname(os.path.abspath(build.__file__)))
    subprocess.run(["python3", "-c", code], check=True, cwd=root, env=dict(os.environ, CXX="/nonexistent/c++"))
