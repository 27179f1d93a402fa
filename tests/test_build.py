"""The build finds the compiler's own HIP headers however the compiler is named (host code, no GPU)."""
import os
import shutil
import subprocess

import pytest

from paper_2602_10940_amd import build

HEADER = os.path.join("hip", "hip_runtime_api.h")


@pytest.mark.parametrize("name", [None, "hipcc", "full"])
def test_hip_headers_are_found_for_a_compiler_named_with_or_without_its_path(name, monkeypatch, tmp_path):
    full = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(full):
        pytest.skip("no hipcc here")
    monkeypatch.setenv("PATH", os.path.dirname(full) + os.pathsep + os.environ["PATH"])
    monkeypatch.chdir(tmp_path)                                   # (a bare name is no path below the current directory)
    if name is None:
        monkeypatch.delenv("HIPCC", raising=False)
    else:
        monkeypatch.setenv("HIPCC", name if name != "full" else full)
    commands = []

    def run(cmd, **kw):
        commands.append(cmd)
        return subprocess.CompletedProcess(cmd, 0, "", "")
    monkeypatch.setattr(build.subprocess, "run", run)
    build._compile_calls()
    (cmd,) = commands
    places = [cmd[i + 1] for i, x in enumerate(cmd) if x == "-isystem"]
    assert any(os.path.isabs(p) and os.path.exists(os.path.join(p, HEADER)) for p in places), places
    assert all(os.path.isdir(p) for p in places if p.endswith("include")), places
