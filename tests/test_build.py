"""The build: the C library first, then the extension module, which is made again when it is older than what it is made from."""
import os
import subprocess
import types

import pytest

from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import build as hip_build


@pytest.fixture
def commands(monkeypatch):
    """What would be run, by its first word; the module's compiler fails if asked to."""
    seen = types.SimpleNamespace(run=[], module_fails=False)

    def run(cmd, **kw):
        seen.run.append(cmd)
        bad = seen.module_fails and cmd[0] != hip_build.HIPCC
        return subprocess.CompletedProcess(cmd, 1 if bad else 0, "", "no Python.h" if bad else "")

    monkeypatch.setattr(hip_build.subprocess, "run", run)
    return seen


def test_the_library_is_built_before_the_module_and_without_it(commands):
    commands.module_fails = True
    with pytest.raises(RuntimeError, match="Python.h"):
        hip_build.build(force=True)
    assert [c[0] == hip_build.HIPCC for c in commands.run] == [True, False]
    assert hip_build.LIB in commands.run[0]


def test_a_module_older_than_its_sources_is_made_again(commands, monkeypatch, tmp_path):
    files = {}
    for name, age in (("module", 10), ("marshal.cpp", 20), ("ts_densify.h", 30)):
        files[name] = str(tmp_path / name)
        open(files[name], "w").close()
        os.utime(files[name], (1e9 - age, 1e9 - age))
    monkeypatch.setattr(hip_build, "MARSHAL", files["module"])
    monkeypatch.setattr(hip_build, "MARSHAL_USES", [files["marshal.cpp"], files["ts_densify.h"]])
    hip_build.build_marshal(force=False)
    assert not commands.run
    for name in ("marshal.cpp", "ts_densify.h"):
        os.utime(files[name], (1e9, 1e9))
        hip_build.build_marshal(force=False)
        assert len(commands.run) == 1
        commands.run.clear()
        os.utime(files[name], (1e9 - 20, 1e9 - 20))
    os.remove(files["module"])
    hip_build.build_marshal(force=False)
    assert len(commands.run) == 1


def test_the_module_belongs_to_this_interpreter():
    import importlib.machinery
    assert ts.MARSHAL_PATH == hip_build.MARSHAL
    assert ts.MARSHAL_PATH.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])
