"""A decode step that fails half way returns only once its copies are done:
their host memory is the step's own, or the caller's.  tests/hip_stub_step.cpp
is linked with the library and stands in for the HIP calls of a step, each of
which fails in turn; nothing here touches a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

asr = pytest.importorskip("paper_2603_11273_amd.asr")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_failed_decode_step_waits_for_its_copies(tmp_path):
    exe = str(tmp_path / "failed_step")
    lib_dir = os.path.dirname(asr.LIB_PATH)
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "hip_stub_step.cpp"), "-L", lib_dir,
           "-l:" + os.path.basename(asr.LIB_PATH), "-Wl,-rpath," + lib_dir,
           "-Wl,--allow-shlib-undefined", "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "failed steps leave nothing pending: ok" in r.stdout
