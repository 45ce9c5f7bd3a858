"""Builds a C++ host test of tests/csrc under the sanitizers and runs it."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host_test(name, tmp_path, sanitizers="address,undefined"):
    exe = str(tmp_path / name)
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer",
                            "-fsanitize=" + sanitizers, "-fno-sanitize-recover=all", "-Wall", "-Wextra", "-Werror",
                            "-I", os.path.join(ROOT, "paper_2307_09226_amd", "csrc"),
                            os.path.join(ROOT, "tests", "csrc", name + ".cpp"), "-o", exe, "-lpthread"],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-4000:]
    assert "ALL OK" in run.stdout
