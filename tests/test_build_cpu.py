"""The build checks that what it built loads, in the interpreter that runs it
(the binding links against that interpreter's PyTorch)."""
import subprocess
import sys

from paper_2609_22870_amd import _build


def test_load_checks_run_this_interpreter(monkeypatch):
    ran = []

    def run(cmd, **kw):
        ran.append(cmd)
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(_build.subprocess, "run", run)
    monkeypatch.setattr(_build.os, "replace", lambda a, b: None)
    _build.build()
    checks = [c for c in ran if "-c" in c and "ctypes.CDLL" in c[c.index("-c") + 1]]
    assert len(checks) == 2 and all(c[0] == sys.executable for c in checks)
