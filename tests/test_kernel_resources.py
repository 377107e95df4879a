"""Registers of the fp32 workgroup backward at D = M = 64: eight waves of 128 registers each.  What does not fit goes to
scratch memory, whose loads wait for the fetch that is under way: with 20 and 12 bytes per lane the kernels were up to 8 %
slower on workgroups of one to three blocks."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_16236_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
@pytest.mark.parametrize("kernel,scratch", [("dq_block_kernel", 8), ("reverse_block_kernel", 0)])
def test_the_fp32_backward_keeps_to_its_registers(tmp_path, kernel, scratch):
    source = tmp_path / "one.hip"
    source.write_text(f'#include "{CSRC}/la_block.h"\nnamespace la {{\n' + "".join(
        f"template __global__ void {kernel}<64, 64, {t}, {s}>(const PassArgs);\n" for t in ("float", "feat_f32") for s in ("false", "true")) + "}\n")
    out = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c", str(source), "-o", str(tmp_path / "one.o")],
                         capture_output=True, text=True, check=True).stderr
    assert [int(x) for x in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", out)] == [4] * 4
    found = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", out)]
    assert len(found) == 4 and max(found) <= scratch, found
