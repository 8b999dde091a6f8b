"""CPU-only checks of the compiled kernels: properties of this library's own gfx950 code that the tile rules and the output path
count on and that no result shows (the pieces an output leaves in, registers that decide how many workgroups a CU holds)."""
import os
import re
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
    for tool in ("llvm-objcopy", "llvm-objdump", "llvm-readelf"):
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


def registers(source, tmp):
    """Kernel name -> (vector registers, spilled ones)."""
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code_object(source, tmp)], capture_output=True, text=True, check=True).stdout
    found = re.findall(r"\.name:\s+(_ZN5nvfp4\S+).*?\.vgpr_count:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)", notes, re.S)
    assert found
    return {name: (int(v), int(s)) for name, v, s in found}


def unwaited_loads(asm):
    """(number of direct-to-LDS loads, the kernels of those whose address registers a lane read wrote fewer than five wait states before)."""
    kernel, before, loads, unwaited = "", [], 0, []
    for line in asm.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:", line)
        if head:
            kernel, before = head.group(1), []
            continue
        ins = line.split("//")[0].strip()
        if not ins:
            continue
        if ins.startswith("global_load_lds"):
            loads += 1
            first, last = map(int, re.search(r"s\[(\d+):(\d+)\]", ins).groups())
            states = 0
            for prev in reversed(before):
                if states >= 5:
                    break
                written = re.match(r"v_read(?:first)?lane_b32 s(\d+)", prev)
                if written and first <= int(written.group(1)) <= last:
                    unwaited.append(kernel)
                    break
                states += int(prev.split()[1]) + 1 if prev.startswith("s_nop") else 1
        before = before[-5:] + [ins]
    return loads, unwaited


def test_unwaited_loads_are_found():
    text = "0000 <k>:\n v_readfirstlane_b32 s1, v3\n s_mov_b32 m0, s28\n s_nop {}\n global_load_lds_dwordx4 v4, s[0:1]\n"
    assert unwaited_loads(text.format(2)) == (1, ["k"]) and unwaited_loads(text.format(3)) == (1, [])


# A scalar register that a vector instruction wrote may be the address of a vector memory instruction five wait states later.  The compiler
# keeps that by itself, but not for the loads in inline assembly, whose own first instructions have to be the wait.
@pytest.mark.parametrize("source", ["quantize", "gemm", "gemm_mx", "gemm_ksplit"])
def test_direct_loads_wait_for_their_address(source, tmp_path):
    asm = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", code_object(source, tmp_path)], capture_output=True, text=True, check=True).stdout
    loads, unwaited = unwaited_loads(asm)
    assert loads > 0 and not unwaited


@pytest.mark.parametrize("source", ["gemm", "gemm_mx", "gemm_ksplit"])
def test_gemm_outputs_leave_in_whole_pieces(source, tmp_path):
    # A 16-byte piece whose store the compiler has split (its last word shared with the form for cut pieces) goes out as 12 + 4 bytes:
    # 5-10 % of a binary32 product.
    asm = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", code_object(source, tmp_path)], capture_output=True, text=True, check=True).stdout
    assert asm.count("global_store_dwordx4") > 0
    assert asm.count("global_store_dwordx3") == 0


def kernels(regs, kind):
    """(template arguments, vector registers, spilled) of the kernels of a kind."""
    for name, (v, s) in regs.items():
        if kind in name:
            yield tuple(int(x or y) for x, y in re.findall(r"Li(\d+)E|Lb(\d)E", name)), v, s


def test_resident_workgroups_of_the_quantizers(tmp_path):
    # 512 registers per SIMD: 128 are four waves, 168 three.  (Three registers above the line cost a columns pass 18 %.)
    regs = registers("quantize", tmp_path)
    seen = 0
    for (dt, b, sf, rnd_r, rnd_c, rpl, src), v, s in kernels(regs, "quantize_dual_kernel"):
        if rpl == 16 and dt == 1 and (b, sf) != (16, 1):
            assert v <= 128 and s == 0, ("dual bf16", b, sf, rnd_r, rnd_c, src, v, s)
            seen += 1
        if rpl == 16 and dt == 0 and rnd_c == 0:
            assert v <= 168 and s <= 2, ("dual f32 RtN", b, sf, v, s)
            seen += 1
        if rpl == 8:
            assert v <= (170 if dt == 0 and sf == 1 else 128) and s == 0, ("dual, 8 rows", dt, b, sf, rnd_r, rnd_c, src, v, s)
    assert seen >= 10
    for (dt, b, sf, rnd, hw, aligned, rpl), v, s in kernels(regs, "quantize_cols_kernel"):
        if rpl == 16 and dt == 1 and hw and aligned and not (b == 16 and sf == 1 and rnd == 0):
            assert v <= 128 and s == 0, ("columns bf16", b, sf, rnd, v, s)
        if rpl == 16 and dt == 0 and hw and rnd == 0 and (b >= 64 or sf == 1):
            assert v <= 168 and s == 0, ("columns f32 RtN", b, sf, v, s)
    for (dt, b, sf, rnd, hw), v, s in kernels(regs, "quantize_rows_kernel"):
        if not (dt == 0 and sf == 1 and rnd == 1):
            assert v <= 64 and s == 0, ("rows", dt, b, sf, rnd, hw, v, s)


def test_resident_workgroups_of_the_streaming_quantizers(tmp_path):
    # three workgroups of four waves per CU: 168 registers
    regs = registers("quantize", tmp_path)
    columns = list(kernels(regs, "quantize_cols_stream_kernel"))
    duals = list(kernels(regs, "quantize_dual_stream_kernel"))
    pairs = list(kernels(regs, "quantize_dual_stream_pair_kernel"))
    assert {a for a, _, _ in columns} == {(16, 0, 0), (16, 0, 1), (16, 1, 1), (32, 0, 0), (32, 0, 1), (32, 1, 0), (32, 1, 1), (64, 0, 1), (64, 1, 1), (128, 0, 1), (128, 1, 1)}
    assert len(duals) == 4 * 3 and {a for a, _, _ in pairs} == {(16, 0), (32, 1)}
    for args, v, s in columns + duals + pairs:
        # (blocks of 16 with E8M0 scales, both sides to nearest: on the line, with ten spilled)
        assert v <= 168 and s <= (10 if args == (16, 1, 0, 0) else 0), (args, v, s)


def test_registers_of_small_tensors_and_four_groups(tmp_path):
    # workgroups of eight waves: two per SIMD need 256 registers (four groups of waves, one workgroup per CU), four 128 (small tensors)
    for args, v, s in kernels(registers("quantize_small", tmp_path), "quantize_small"):
        assert v <= 128 and s == 0, (args, v, s)
    four = [(args, v, s) for args, v, s in kernels(registers("gemm", tmp_path), "gemm_nt_f16_kernel") if args[5] == 4]
    assert len(four) == 4 * 2 * 2 * 2  # (blocks, tiles, output types, K tail)
    for (block, wm, wn, ta, tb, groups, out, tail), v, s in four:
        assert v <= 256 and s == 0, (block, ta, out, tail, v, s)
    # eight waves of 96 and 64 rows: two per SIMD as well
    uneven = list(kernels(registers("gemm", tmp_path), "gemm_nt_f16_uneven_kernel"))
    assert len(uneven) == 4 * 2 * 2  # (blocks, output types, K tail)
    for args, v, s in uneven:
        assert v <= 256 and s == 0, (args, v, s)
    # (128 x 256 in two groups is a tile of the kernels of four waves alone: test_products_of_one_wave_per_simd)
    assert not [args for args, v, s in kernels(registers("gemm", tmp_path), "gemm_nt_f16_kernel") if args[5] == 2]
    assert [args for args, v, s in kernels(registers("gemm_wide16", tmp_path), "gemm_nt_f16_wide_kernel") if args[3] == 2]


def test_rows_of_small_tensors_bring_little_along(tmp_path):
    # 2 us of row quantization: with the LDS and the four jobs of the kernel for both orientations, decode calls took 0.4 us longer
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code_object("quantize_small", tmp_path)], capture_output=True, text=True, check=True).stdout
    rows = [int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", k).group(1)) for k in notes.split("  - .agpr_count") if "quantize_small_rows" in k]
    assert len(rows) == 2 * 4 * 3  # (element types, formats; round to nearest, stochastic, two tensors)
    assert max(rows) <= 1024


def test_few_rows_kernels(tmp_path):
    # the direct loads' waits as above; workgroups of 16 waves, four per SIMD: 128 registers
    asm = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", code_object("gemm_thin", tmp_path)], capture_output=True, text=True, check=True).stdout
    loads, unwaited = unwaited_loads(asm)
    assert loads > 0 and not unwaited
    thin = list(kernels(registers("gemm_thin", tmp_path), "gemm_nt_thin_kernel"))
    assert len(thin) == 3 * 2 * 7 * 2  # (A packed, binary32, bf16; formats; tiles; output types)
    for args, v, s in thin:
        assert v <= 128 and s == 0, (args, v, s)


def test_fused_layers_registers(tmp_path):
    # workgroups of eight waves, one per CU: 256 registers
    fused = list(kernels(registers("fused_small", tmp_path), "small_"))
    assert len(fused) == 2 * 2 * 2 * 2  # (directions, element types, formats, output types)
    for args, v, s in fused:
        assert v <= 256 and s == 0, (args, v, s)


def test_registers_of_the_mxfp4_products(tmp_path):
    # four waves of 128 x 128, one per SIMD, on all 512 registers: seven spilled cost an MXFP4 step 1 %; the other tiles run two waves per SIMD
    regs = registers("gemm_mx", tmp_path)
    direct, tile = list(kernels(regs, "gemm_nt_mxfp4_dma_kernel")), list(kernels(regs, "gemm_nt_mxfp4_tile_kernel"))
    assert len(direct) == 2 * 4 and len(tile) == 2 * 3  # (output types; layouts, tiles)
    for args, v, s in direct + tile:
        assert v <= (512 if len(args) == 3 else 256) and s == 0, (args, v, s)


def test_arguments_of_the_products(tmp_path):
    # a launch's arguments are copied by the host: 16 bytes more than 196 cost calls that are bound by its work up to 0.3 us (launch_gemm())
    for source, most in (("gemm", 104), ("gemm_mx", 104), ("gemm_ksplit", 196)):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code_object(source, tmp_path)], capture_output=True, text=True, check=True).stdout
        sizes = [int(n) for n in re.findall(r"\.kernarg_segment_size:\s+(\d+)", notes)]
        assert sizes and max(sizes) <= most, source


def late_operands(asm):
    """(number of matrix instructions on accumulators of the AGPRs, the kernels of those of which a vector instruction wrote an operand less than
    two wait states before)."""
    kernel, before, found, late = "", [], 0, []
    span = lambda t: (lambda m: set(range(int(m.group(1)), int(m.group(2) or m.group(1)) + 1)) if m else set())(re.fullmatch(r"v\[?(\d+)(?::(\d+)\])?", t.strip()))
    for line in asm.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:", line)
        if head:
            kernel, before = head.group(1), []
            continue
        ins = line.split("//")[0].strip()
        if not ins:
            continue
        if ins.startswith("v_mfma") and " a[" in ins:
            found += 1
            operands = set().union(*(span(t) for t in re.findall(r"v\[\d+:\d+\]|\bv\d+\b", ins.split(" ", 1)[1])))
            states = 0
            for prev in reversed(before):
                if states >= 2:
                    break
                if prev.startswith("v_") and not prev.startswith("v_mfma") and span(prev.split(" ", 1)[1].split(",")[0]) & operands:
                    late.append(kernel)
                    break
                states += int(prev.split()[1]) + 1 if prev.startswith("s_nop") else 1
        before = before[-3:] + [ins]
    return found, late


def test_late_operands_are_found():
    text = "0000 <k>:\n v_pk_mul_f16 v7, v3, v2\n{} v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[0:3]\n"
    assert late_operands(text.format(" s_add_u32 s0, s0, s1\n")) == (1, ["k"]) and late_operands(text.format(" s_nop 1\n")) == (1, [])


# The matrix instructions of the kernels with one wave per SIMD are inline assembly, so the compiler does not keep their operands' wait states, nor those of
# the direct loads' addresses.  512 registers, none spilled; outputs in whole pieces, as above.
@pytest.mark.parametrize("source", ["gemm_wide16", "gemm_wide32", "gemm_wide64", "gemm_wide128", "gemm_mx"])
def test_products_of_one_wave_per_simd(source, tmp_path):
    asm = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", code_object(source, tmp_path)], capture_output=True, text=True, check=True).stdout
    loads, unwaited = unwaited_loads(asm)
    found, late = late_operands(asm)
    assert loads > 0 and not unwaited and found > 0 and not late and asm.count("global_store_dwordx3") == 0
    for args, v, s in kernels(registers(source, tmp_path), "wide" if source != "gemm_mx" else "gemm_nt_mxfp4_dma_kernel"):
        assert v <= 512 and s == 0, (args, v, s)
