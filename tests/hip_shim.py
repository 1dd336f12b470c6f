"""Runs a test's program in a process of its own, where a small library comes
before the HIP runtime: functions that it defines are the ones that the library
calls."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2311_12281_amd import build as B


def run_child(tmp_path, shim, program, timeout=100):
    """The program gets the path of the compiled shim as its argument, loads it globally before the
    package, and prints OK at its end."""
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, so, child = tmp_path / "shim.cpp", tmp_path / "shim.so", tmp_path / "child.py"
    src.write_text(shim)
    child.write_text(program)
    subprocess.run([cxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    env = dict(os.environ, PYTHONPATH=B.ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    r = subprocess.run([sys.executable, "-u", str(child), str(so)], cwd=B.ROOT, env=env, capture_output=True, text=True,
                       timeout=timeout)
    assert r.returncode == 0 and r.stdout.endswith("OK\n"), r.stdout[-1000:] + r.stderr[-2000:]
