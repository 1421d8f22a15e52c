"""The library and the Python layer do without the native marshalling (csrc/marshal.cpp): the build makes the library where there is no torch
or no headers, and calls whose extension is missing, damaged or made for another Python or torch are checked in Python."""
import os
import shutil
import stat
import subprocess
import sys

import pytest
import torch

from paper_2605_11005_amd import binding as B

CSRC = os.path.join(os.path.dirname(os.path.abspath(B.__file__)), "csrc")


def _tool(path, body):
    path.write_text("#!/bin/bash\n" + body)
    path.chmod(path.stat().st_mode | stat.S_IXUSR)


@pytest.mark.parametrize("missing", ["torch", "headers", "nothing"])
def test_the_library_is_built_without_the_marshalling(missing, tmp_path):
    package, tools = tmp_path / "package", tmp_path / "tools"
    (package / "csrc").mkdir(parents=True)
    tools.mkdir()
    shutil.copy(os.path.join(CSRC, "build.sh"), package / "csrc")
    writes_its_output = 'while [ "$1" != -o ]; do shift; done; touch "$2"\n'
    _tool(tools / "hipcc", writes_its_output)
    _tool(tools / "g++", "exit 1\n" if missing == "headers" else writes_its_output)
    _tool(tools / "python", "exit 1\n" if missing == "torch" else f'exec {sys.executable} "$@"\n')
    env = dict(os.environ, PATH=f"{tools}:{os.environ['PATH']}", PYTHON=str(tools / "python"))
    subprocess.run(["bash", str(package / "csrc" / "build.sh")], check=True, env=env)
    built = {f.name for f in package.iterdir()} - {"csrc"}
    assert built == {"libmoe_mi355x.so"} | ({os.path.basename(B.marshal_path())} if missing == "nothing" else set())


@pytest.mark.parametrize("damage", ["missing", "damaged"])
def test_calls_are_checked_in_python_without_the_marshalling(damage, tmp_path, monkeypatch):
    path = tmp_path / "_marshal.so"
    if damage == "damaged":
        path.write_bytes(b"\x7fELF of something else")
    monkeypatch.setattr(B, "_MARSHAL", None)
    monkeypatch.setattr(B, "marshal_path", lambda: str(path))
    t = torch.zeros((4, 8))
    with pytest.warns(RuntimeWarning, match="native marshalling"), pytest.raises(B.MoeError, match="contiguous device tensor"):
        B.moe_route(t, 2, 0, 0, 8, t, t, t)
