"""CPU-only checks of outputs that two kinds of tiles share: which products take one, and that the tiles cover every output once."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

from paper_2505_19115_amd import binding as nv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
E4M3_64 = nv.Format(64, nv.SCALE_E4M3, 1)


def products(n):
    rng = random.Random(5)
    for _ in range(n):
        yield rng.randrange(256, 14000), rng.randrange(256, 14000), 128 * rng.randrange(8, 90)


def test_which_products_mix_tiles():
    kinds = set()
    for M, N, K in products(4000):
        mix, tiles = nv.gemm_mixed(M, N, K), -(-M // 256) * -(-N // 256)
        assert mix == nv.gemm_mixed(M, N, K, E4M3_64) and nv.gemm_mixed(M, N, K, nv.MXFP4) is None
        if mix is None:
            continue
        # 256 x 256 by the rule, at least 18 whole K tiles, a last round that is not full; whole rounds of the first kind, one of the second
        assert nv.gemm_tile(M, N, K) == (256, 256) and K >= 18 * 128 and tiles > 256 and tiles % 256
        whole = (tiles - 1) // 256 * 256
        assert 0 < mix["first"] <= whole and mix["first"] + mix["second"] <= whole + 256
        kinds.add((mix["rows"], mix["tile"], mix["groups"]))
    assert kinds == {(r, t, g) for r in (False, True) for t, g in (((192, 256), 1), ((128, 256), 2))}
    for M, N, K in ((4096, 11008, 2176), (4096, 11008, 4096 + 32), (4096, 4096, 11008), (0, 11008, 4096), (4096, 11008, -4096)):
        assert nv.gemm_mixed(M, N, K) is None
    assert nv.gemm_mixed(4096, 11008, 4096) == dict(rows=False, split=32, first=512, second=242, tile=(192, 256), groups=1)
    assert nv.gemm_mixed(4096, 11008, 4096, nv.Format(8, nv.SCALE_E4M3, 1)) is None
    f = nv.NVFP4.c()
    assert nv.lib.nvfp4_host_gemm_mixed(4096, 11008, 4096, C.byref(f), None) == 0 and nv.lib.nvfp4_host_gemm_mixed(4096, 11008, 4096, None, (C.c_int32 * 7)()) == 0


@pytest.mark.skipif(not shutil.which(CLANG), reason="needs the ROCm compilers")
def test_every_output_belongs_to_one_tile(tmp_path):
    exe = str(tmp_path / "mixed_tiles")
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wno-unknown-pragmas", "-o", exe, os.path.join(ROOT, "tests", "mixed_tiles_main.cpp")])
    lines = []
    for M, N, K in products(4000):
        mix = nv.gemm_mixed(M, N, K)
        if mix:
            lines.append(f"{M} {N} {int(mix['rows'])} {mix['split']} {mix['first']} {mix['second']} {mix['tile'][0]}")
    assert len(lines) > 300
    p = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and f"mixed-tiles ok {len(lines)}" in p.stdout, p.stderr
