"""CPU-only checks of the compiled kernels: properties of this library's own gfx950 code that no result shows."""
import os
import shutil
import struct
import subprocess

import pytest

from paper_2505_19115_amd import build as hip_build

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_object(source: str, tmp) -> str:
    """The gfx950 code object inside the object file that build() compiled from a source, as a file of its own."""
    obj = os.path.join(hip_build.OBJ, source + ".o")
    for tool in ("llvm-objcopy", "llvm-objdump"):
        if not shutil.which(os.path.join(LLVM, tool)):
            pytest.skip(f"{tool} is not installed")
    if not os.path.exists(obj):
        pytest.skip(f"{obj} is not there (build() makes it)")
    fat = str(tmp / (source + ".fatbin"))
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", obj, str(tmp / "unused.o")])
    data = open(fat, "rb").read()
    at = data.index(MAGIC)
    pos = at + len(MAGIC) + 8
    for _ in range(struct.unpack_from("<Q", data, at + len(MAGIC))[0]):
        offset, size, name_len = struct.unpack_from("<QQQ", data, pos)
        name = data[pos + 24:pos + 24 + name_len]
        pos += 24 + name_len
        if b"gfx950" in name:
            out = str(tmp / (source + ".co"))
            open(out, "wb").write(data[at + offset:at + offset + size])
            return out
    raise AssertionError("no gfx950 code object")


@pytest.mark.parametrize("source", ["gemm", "gemm_mx", "gemm_ksplit"])
def test_gemm_outputs_leave_in_whole_pieces(source, tmp_path):
    # A 16-byte piece whose store the compiler has split (its last word shared with the form for cut pieces) goes out as 12 + 4 bytes:
    # 5-10 % of a binary32 product.
    asm = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", code_object(source, tmp_path)], capture_output=True, text=True, check=True).stdout
    assert asm.count("global_store_dwordx4") > 0
    assert asm.count("global_store_dwordx3") == 0
