"""CPU-only walk of the direct-to-LDS MXFP4 kernel's loads (csrc/mx_codes.h): none leaves its operand, and that the kernel takes every address
of an operand's codes from there."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"


@pytest.mark.skipif(not shutil.which(CLANG), reason="needs the ROCm compilers")
def test_loads_of_codes_stay_inside_their_operand(tmp_path):
    exe = str(tmp_path / "mx_codes")
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wno-unknown-pragmas", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-o", exe, os.path.join(ROOT, "tests", "mx_codes_main.cpp")])
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and "mx-codes ok" in p.stdout, p.stderr


def test_the_kernel_aims_an_operands_loads_at_that_operand():
    src = open(os.path.join(ROOT, "paper_2505_19115_amd", "csrc", "gemm_mx.hip")).read()
    body = src[src.index("gemm_nt_mxfp4_dma_kernel(TileArgs P)"):src.index("#undef NVFP4_MXD_LOAD_B")]
    for x in "AB":
        assert len(re.findall(rf"\b{x}\.past_end\(\)", body)) == 1 and len(re.findall(rf"\b{x}\.start\(.*P\.{x}_codes.*P\.{x}_codes", body)) == 1
        assert re.search(rf"#define NVFP4_MXD_LOAD_{x}\(u\) NVFP4_MXD_LOAD\({x}\.off\[.*\], {x}\.p, {x}\.more\(u\)\)", body)
        assert not re.search(rf"\b{x}\.(p|tile|step|off\[[^\]]*\])\s*[-+]?=[^=]", body)
