"""The small-batch tiles' forms on the host (no GPU): csrc/decode_form.h picks
how many one-wave workgroups of a launch share a CU and gives each its LDS.
tests/native/decode_form_check.cpp compiles that header for the host.  The
registers are those of the built library's kernels."""

import os
import shutil
import subprocess

import pytest

from tests.kernel_resources import VGPRS_PER_LANE, kernels

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


ROOM, SIX = 1, 6  # DecodeForm: P's form beside D's layers, D's beside P's small tiles


def test_a_d_tile_fits_beside_waiting_p_tiles():
    """P's workgroups of the form that leaves room fit on a CU four times, so one
    to a SIMD or some SIMD has none: a SIMD's registers hold one of P's and one
    of D's waves, whichever GEMM either is in."""
    got = kernels()
    bf16 = ("gemm1_swiglu_decode<false, {}>", "gemm1_swiglu_decode<true, {}>", "gemm2_down_decode<false, {}>",
            "gemm2_down_decode<true, {}>")
    mx = tuple(f"gemm_mx_skinny<{gated}, {sc4}, {{}}>" for gated in ("true", "false") for sc4 in ("true", "false"))
    for names in (bf16, mx):
        p = max(got[n.format(ROOM)][0] for n in names)
        d = max(got[n.format(SIX)][0] for n in names)
        assert p + d <= VGPRS_PER_LANE, (p, d)
