"""The library's host-side rules (which kernel a call takes, where its scratch
lies), checked on the CPU by tests/host/route_check.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_routes_and_layout(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "route_check")
    r = subprocess.run([cc, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "paper_0904_1179_amd", "csrc", "layout.cpp"),
                        os.path.join(ROOT, "tests", "host", "route_check.cpp")],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("0 failures"), r.stdout + r.stderr
