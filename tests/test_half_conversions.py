"""The library's device code holds no FP16 conversion folded into a multiply-add:
v_fma_mixlo_f16 and v_fma_mixhi_f16 round once where the FP32 result is to be
rounded and then converted, as a store and a load do."""
import os
import shutil
import subprocess

import pytest

from paper_1307_4703_amd import build_lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
@pytest.mark.skipif(not os.path.exists(build_lib.OUT), reason="library not built")
def test_no_folded_half_conversion(tmp_path):
    lib = str(tmp_path / "libgg.so")
    shutil.copy(build_lib.OUT, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objs = sorted(f for f in os.listdir(tmp_path) if "gfx950" in f)
    assert objs, "no device code found"
    found, packed = [], 0
    for f in objs:
        text = subprocess.run([OBJDUMP, "-d", str(tmp_path / f)], check=True, capture_output=True,
                              text=True).stdout
        packed += text.count("v_cvt_pk_f16_f32") + text.count("v_cvt_f16_f32")
        kernel = ""
        for line in text.splitlines():
            if line.endswith(">:"):
                kernel = line
            elif "v_fma_mixlo_f16" in line or "v_fma_mixhi_f16" in line:
                found.append((f, kernel))
    assert packed > 0
    assert not found, found[:4]
