"""The small-batch tiles' forms on the host (no GPU): csrc/decode_form.h picks
how many one-wave workgroups of a launch share a CU and gives each its LDS.
tests/native/decode_form_check.cpp compiles that header for the host.  The
registers are those of the built library's kernels."""

import os
import shutil
import subprocess

import pytest

from synth import BF16, FP8
from tests import test_gpu_decode_forms as forms
from tests.kernel_resources import LDS_UNITS, VGPRS_PER_LANE, kernels, lds_units

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


def test_d_small_kernels_fit_beside_fp8_ring_tiles():
    """P's FP8 ring tiles of up to 192 rows leave a SIMD the registers of D's route,
    permute and combine waves, and a CU some LDS (the taller ones take it all)."""
    got = kernels()
    small = max(v[0] for k, v in got.items()
                if k.startswith(("route_kernel", "permute_mx_kernel", "combine_kernel<2, 2")))
    for gemm in (1, 2):
        for sc4 in ("false", "true"):
            vgprs, lds = got[f"gemm{gemm}_mx_prefill<{sc4}, false>"]
            assert vgprs + small <= VGPRS_PER_LANE, (gemm, sc4, vgprs, small)
            assert lds_units(lds) < LDS_UNITS, (gemm, sc4, lds)


def _form(check, E, e_loc, k, T, n_tiles):
    r = subprocess.run([check, "form"] + [str(v) for v in (E, e_loc, k, T, n_tiles)], stdout=subprocess.PIPE, text=True,
                       timeout=60)
    return int(r.stdout)


def _n_tiles(dtype, H, I):
    """Column tiles of a launch of staged tiles: GEMM1's are 32 columns of gate
    and up, GEMM2's 64 columns, 32 for bf16 with a rotated K."""
    rot = dtype == BF16 and I % 2048 == 0
    return I // 32, H // (32 if rot else 64)


def test_gpu_shapes_take_the_forms_they_name(check):
    """The edge rows of the GPU test run in every form that a launch by its tile
    count can take: each type, GEMM, and K order or scale gather, four, six and
    eight workgroups per CU; the FP8 ones are compared with four."""
    seen = set()
    for dtype, H, I, form1, form2 in forms.SHAPES:
        n1, n2 = _n_tiles(dtype, H, I)
        got = [_form(check, forms.E, forms.E_LOC, 1, forms.T, n) for n in (n1, n2)]
        assert got == [form1, form2], (dtype, H, I, got)
        special = (H % 2048 == 0, I % 2048 == 0) if dtype == BF16 else (H % 512 == 0, I % 512 == 0)
        seen |= {(dtype, gemm, special[gemm], got[gemm]) for gemm in (0, 1)}
        if dtype == FP8:
            assert [_form(check, forms.E_FOUR, forms.E_LOC, 1, forms.T, n) for n in (n1, n2)] == [4, 4], (H, I)
    assert seen == {(d, gemm, s, f) for d in (BF16, FP8) for gemm in (0, 1) for s in (False, True) for f in (4, 6, 8)}
