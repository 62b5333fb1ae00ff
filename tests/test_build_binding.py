"""The native call marshalling is used with the torch and Python it was built for only, and built anew for others (CPU)."""
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
