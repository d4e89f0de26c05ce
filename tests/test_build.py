"""The library's build: it needs no torch, and the extension module of the Python binding can fail without taking it along."""
import os
import subprocess
import sys

import pytest

from paper_2604_18616_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def fake(tmp_path, monkeypatch):
    """A build into a folder of its own whose compiler only writes the file it is asked for."""
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "NATIVE_PATH", str(tmp_path / "module.so"))
    commands = []

    def run(cmd, verbose):
        commands.append(cmd)
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write(cmd[-1])
    monkeypatch.setattr(build, "_run", run)
    return tmp_path, commands


def test_library_and_module_are_built(fake, monkeypatch):
    folder, commands = fake
    assert build.build_library() == str(folder / "lib.so")
    assert sorted(os.listdir(folder)) == ["lib.so", "module.so", "obj"]
    assert len(commands) == len(build.SOURCES) + 2
    del commands[:]
    build.build_library(incremental=True)
    assert len(commands) == 1                            # the link
    build.build_library()
    assert len(commands) == 1 + len(build.SOURCES) + 2
    del commands[:]
    newer = os.path.getmtime(folder / "module.so") + 10
    monkeypatch.setattr(build, "_newest_header", lambda: newer)
    build.build_library(incremental=True)
    assert len(commands) == len(build.SOURCES) + 2       # a header is newer
    monkeypatch.undo()


def test_the_module_is_made_again_for_another_torch(fake, monkeypatch):
    import torch
    folder, commands = fake
    build.build_library()
    del commands[:]
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".1")
    build.build_library(incremental=True)
    assert len(commands) == 2                            # the link, and the module for the other torch


@pytest.mark.parametrize("why", [ImportError("no torch"), RuntimeError("hipcc failed")])
def test_a_module_that_cannot_be_built_leaves_the_library(fake, monkeypatch, why):
    folder, commands = fake
    (folder / "module.so").write_text("of an older library")
    run = build._run

    def fail(cmd, verbose):
        run(cmd, verbose)
        if cmd[cmd.index("-o") + 1].startswith(str(folder / "module.so")):
            raise why
    if isinstance(why, ImportError):
        def no_torch(out):
            raise why
        monkeypatch.setattr(build, "_native_command", no_torch)
    else:
        monkeypatch.setattr(build, "_run", fail)
    with pytest.warns(UserWarning, match=str(why)):
        assert build.build_library() == str(folder / "lib.so")
    assert sorted(os.listdir(folder)) == ["lib.so", "obj"]


def test_a_library_that_cannot_be_built_raises(fake, monkeypatch):
    folder, commands = fake

    def fail(cmd, verbose):
        raise RuntimeError("hipcc failed")
    monkeypatch.setattr(build, "_run", fail)
    with pytest.raises(RuntimeError, match="hipcc failed"):
        build.build_library()
    assert os.listdir(folder) == ["obj"]


def test_build_without_torch(tmp_path):
    """In a process that cannot import torch, with a compiler that only writes files."""
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\n: > "$2"\n')
    hipcc.chmod(0o755)
    code = ("import sys, warnings; sys.modules['torch'] = None; sys.path.insert(0, sys.argv[1])\n"
            "import importlib.util as u\n"
            "spec = u.spec_from_file_location('build', sys.argv[1] + '/build.py'); b = u.module_from_spec(spec); spec.loader.exec_module(b)\n"
            "t = sys.argv[2]; b.OBJ_DIR, b.LIB_PATH, b.NATIVE_PATH = t + '/obj', t + '/lib.so', t + '/module.so'\n"
            "warnings.simplefilter('ignore'); print(b.build_library())\n")
    done = subprocess.run([sys.executable, "-c", code, os.path.dirname(build.__file__), str(tmp_path)], env=dict(os.environ, HIPCC=str(hipcc)),
                          stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    assert done.returncode == 0 and os.path.exists(tmp_path / "lib.so") and not os.path.exists(tmp_path / "module.so"), done.stdout
