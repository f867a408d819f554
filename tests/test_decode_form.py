"""The small-batch tiles' forms on the host (no GPU): csrc/decode_form.h picks
how many one-wave workgroups of a launch share a CU and gives each its LDS.
tests/native/decode_form_check.cpp compiles that header for the host."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_00993_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("decode_form") / "decode_form_check")
    cmd = [cxx, "-O1", "-std=c++17", f"-I{CSRC}", os.path.join(ROOT, "tests", "native", "decode_form_check.cpp"), "-o",
           exe]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, f"build failed:\n{' '.join(cmd)}\n{p.stdout}"
    return exe


def test_forms_fit_a_cu(check):
    r = subprocess.run([check], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout
