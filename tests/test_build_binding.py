"""The native call marshalling is used with the torch and Python it was built for only, and built anew for others; the library does not need it (CPU)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def build(monkeypatch):
    import paper_2009_13062_amd.build as build
    if not os.path.exists(build.BINDING):
        pytest.skip("no binding built here")
    return build


def _native_with(setup):
    return subprocess.run([sys.executable, "-c", "import torch; %s; import paper_2009_13062_amd as nf; print(nf._native is not None)" % setup],
                          cwd=ROOT, capture_output=True, text=True, check=True).stdout.split()[-1]


def test_not_used_with_another_torch(build):
    assert _native_with("pass") == "True"
    assert _native_with("torch.__version__ = '2.99.0'") == "False"
    assert _native_with("torch.version.git_version = '0'") == "False"


def test_built_anew_for_another_torch(build, monkeypatch):
    import torch
    ran = []
    monkeypatch.setattr(build.subprocess, "check_call", lambda cmd: ran.append(cmd))
    monkeypatch.setattr(build.os, "replace", lambda a, b: None)
    monkeypatch.setattr(build.os.path, "getmtime", lambda p: float(p == build.BINDING))
    build._build_binding(False, force=False)
    assert not ran
    monkeypatch.setattr(torch, "__version__", "2.99.0")
    build._build_binding(False, force=False)
    assert len(ran) == 1


def _build_without(build, monkeypatch, tmp_path, result):
    """Everything but the library's link replaced: what build() does when the binding ends in `result`."""
    ran = []

    def check_call(cmd):
        ran.append(cmd[0])
        if cmd[0] == "g++":
            raise result
    monkeypatch.setattr(build.subprocess, "check_call", check_call)
    monkeypatch.setattr(build, "_compile", lambda s, *a: s)
    monkeypatch.setattr(build.os, "replace", lambda a, b: None)
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    return ran


def test_the_library_is_built_without_a_host_compiler(build, monkeypatch, tmp_path):
    ran = _build_without(build, monkeypatch, tmp_path, FileNotFoundError("g++"))
    monkeypatch.setattr("shutil.which", lambda name: None)
    with pytest.warns(UserWarning, match="marshalled in Python"):
        build.build()
    assert ran == [build._hipcc()]


def test_a_binding_that_does_not_compile_is_an_error_after_the_library(build, monkeypatch, tmp_path):
    ran = _build_without(build, monkeypatch, tmp_path, subprocess.CalledProcessError(1, "g++"))
    with pytest.raises(subprocess.CalledProcessError):
        build.build()
    assert build._hipcc() in ran
