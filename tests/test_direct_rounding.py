"""The direct kernels round f32 toward minus infinity for a wave's whole life, so
nothing in them but the requantiser may be worked out in f32.  The compiler
turns a division by a run-time value into a reciprocal and conversions: its
assembly of one kernel of each kind must hold none."""
import os
import re
import subprocess

import pytest

from paper_2202_06819_amd import build

KERNELS = {   # BITS, FKB, NP, FP, EXT, LA, MULTI, LIN, WRES, B16
    "depth": "8, 2, 2, 2, true, 3, true, false, false, false",
    "depth_1x1": "4, 4, 2, 4, false, 4, true, true, false, false",
    "resident": "4, 2, 2, 2, true, 3, true, false, true, false",
    "resident_1x1": "8, 4, 2, 2, true, 4, true, true, true, false",
}


@pytest.mark.parametrize("kind", KERNELS)
def test_no_division_in_f32(kind, tmp_path):
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "qconv_direct.h"\nnamespace qconv {\n'
                   f"template __global__ void conv_direct<{KERNELS[kind]}>(DirectArgs);\n}}\n")
    subprocess.run([build._hipcc(), *build.CFLAGS, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    assert re.search(r"s_setreg_imm32_b32 hwreg\(HW_REG_MODE, 0, 2\), 2", text)
    assert "v_mfma_i32_16x16x64_i8" in text and "v_cvt_pk_u8_f32" in text
    found = sorted(set(re.findall(r"\bv_(?:rcp|rsq|div|sqrt|exp|log)\w*|\bv_cvt_u32_f32\w*", text)))
    assert not found, f"f32 arithmetic beside the requantiser: {found}"
