"""CPU-only checks of the HIP library's host side: the shared object loads and exports the
declared C ABI, argument validation returns the documented codes before anything is launched,
and the scalar steps the kernels use (compiled for the host) agree with the oracle."""
import ctypes as C
import os
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2505_19115_amd import binding as nv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _p(a):
    return a.ctypes.data_as(C.c_void_p)


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "nvfp4.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(nvfp4_[a-z0-9_]+)\s*\(", hdr))
    assert len(declared) >= 20
    raw = C.CDLL(nv.LIB_PATH)
    for name in declared:
        assert hasattr(raw, name), name
    assert declared == set(nv.EXPORTS)


def test_stream_handle(monkeypatch):
    # the current device's current stream, also from a torch without the raw handle; a process without a GPU gets torch's own error
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("Stream", (), {"cuda_stream": 7}))
    monkeypatch.setattr(nv, "_raw_device", lambda: 3)
    monkeypatch.setattr(nv, "_raw_stream", lambda device: 100 + device)
    assert nv._stream() == 103
    for lacking in ("_raw_device", "_raw_stream"):
        with monkeypatch.context() as m:
            m.setattr(nv, lacking, None)
            assert nv._stream() == 7
    monkeypatch.undo()
    if not torch.cuda.is_available():
        with pytest.raises((RuntimeError, AssertionError), match="GPU|HIP|CUDA"):
            nv._stream()


def test_sizes():
    f = nv.NVFP4.c()
    assert nv.lib.nvfp4_codes_bytes(8192, 8192) == 8192 * 8192 // 2
    assert nv.lib.nvfp4_scales_bytes(8192, 4096, 1, C.byref(f)) == 8192 * 4096 // 16
    assert nv.lib.nvfp4_scales_bytes(8192, 4096, 0, C.byref(f)) == 4096 * 8192 // 16
    m = nv.MXFP4.c()
    assert nv.lib.nvfp4_scales_bytes(64, 128, 1, C.byref(m)) == 64 * 4
    assert nv.lib.nvfp4_quantize_workspace_bytes(10, 10) >= 4
    fw = nv.lib.nvfp4_linear_fwd_workspace_bytes(4096, 11008, 4096, C.byref(f))
    assert fw >= (4096 + 11008) * 4096 * 9 // 16
    bw = nv.lib.nvfp4_linear_bwd_workspace_bytes(4096, 11008, 4096, C.byref(f))
    assert bw >= 2 * 4096 * 11008 * 9 // 16 + (4096 + 11008) * 4096 * 9 // 16
    assert nv.lib.nvfp4_status_string(0) == b"ok"
    for code in range(1, 7):
        assert len(nv.lib.nvfp4_status_string(code)) > 3


FAKE = 0x10000  # non-null, 16-byte aligned; never dereferenced because validation fails first


def _quant(x=FAKE, dt=nv.BF16, rows=64, cols=64, ld=64, axis=1, rnd=nv.RTN, fmt=nv.NVFP4,
           codes=FAKE, scales=FAKE, ts=FAKE, flags=0, ws=FAKE, ws_bytes=1 << 20):
    f = fmt.c()
    return nv.lib.nvfp4_quantize(x, dt, rows, cols, ld, axis, rnd, 0, C.byref(f), codes, scales, ts,
                                 flags, ws, ws_bytes, None)


def test_quantize_argument_errors():
    assert _quant(x=None) == nv.EINVAL
    assert _quant(codes=None) == nv.EINVAL
    assert _quant(dt=7) == nv.EINVAL
    assert _quant(axis=2) == nv.EINVAL
    assert _quant(rnd=3) == nv.EINVAL
    assert _quant(flags=8) == nv.EINVAL
    assert _quant(rows=-1) == nv.ESHAPE
    assert _quant(cols=72, ld=72) == nv.ESHAPE            # 72 is not a multiple of 16
    assert _quant(rows=24, axis=0) == nv.ESHAPE           # blocked axis is rows
    assert _quant(ld=32) == nv.ESHAPE                     # ld < cols
    assert _quant(x=FAKE + 2) == nv.EALIGN
    assert _quant(ld=68) == nv.EALIGN                     # rows not 16-byte aligned (bf16)
    assert _quant(fmt=nv.Format(8, 0, 1)) == nv.EUNSUPPORTED
    assert _quant(fmt=nv.Format(32, nv.SCALE_E8M0, 1)) == nv.EUNSUPPORTED
    assert _quant(fmt=nv.Format(16, 5, 1)) == nv.EINVAL
    assert _quant(ws=None) == nv.EWORKSPACE
    assert _quant(ws_bytes=2) == nv.EWORKSPACE


def test_quantize_static_argument_errors():
    # the entry that allocates nothing validates like nvfp4_quantize, and refuses a tensor whose partial maxima
    # do not fit its static scratch before it touches any device
    def qs(x=FAKE, rows=64, cols=64, ld=64, axis=1, rnd=nv.RTN, fmt=nv.NVFP4, codes=FAKE, ts=FAKE, flags=0):
        f = fmt.c()
        return nv.lib.nvfp4_quantize_static(x, nv.BF16, rows, cols, ld, axis, rnd, 0, C.byref(f), codes, FAKE, ts, flags, None)
    assert qs(rows=16385, cols=16, ld=24) == nv.EWORKSPACE          # 16385 row spans > 16384 partial maxima
    assert qs(rows=4096, cols=5 * 8192, ld=5 * 8192 + 8) == nv.EWORKSPACE
    assert qs(rows=16385, cols=16, ld=24, flags=nv.PRESET_TSCALE) == nv.EWORKSPACE  # the limit does not depend on flags


def test_weight_operand_argument_errors():
    f = nv.NVFP4.c()
    n = nv.lib.nvfp4_weight_operands_bytes(11008, 4096, C.byref(f))
    assert n >= 2 * 11008 * 4096 * 9 // 16 and n < 2 * 11008 * 4096 * 9 // 16 + (1 << 21)
    assert nv.lib.nvfp4_weight_operands_bytes(0, 4096, C.byref(f)) == 0
    qw = lambda **k: nv.lib.nvfp4_quantize_weight(k.get("W", FAKE), k.get("dt", nv.BF16), k.get("M", 256), k.get("N", 128), k.get("K", 128),
                                                  C.byref(k.get("f", f)), k.get("out", FAKE + 256 - FAKE % 256 if FAKE % 256 else FAKE), k.get("ws", FAKE), k.get("wsb", 1 << 20), None)
    assert qw(W=None) == nv.EINVAL
    assert qw(out=None) == nv.EINVAL
    assert qw(dt=5) == nv.EINVAL
    assert qw(N=72) == nv.ESHAPE          # W^T is blocked along N
    assert qw(K=48) == nv.ESHAPE
    assert qw(M=0) == nv.ESHAPE
    assert qw(out=FAKE + 16) == nv.EALIGN
    assert qw(ws=None) == nv.EWORKSPACE
    assert qw(f=nv.Format(64, nv.SCALE_E8M0, 0).c()) == nv.EUNSUPPORTED
    fw = lambda **k: nv.lib.nvfp4_linear_fwd_wq(FAKE, k.get("wq", FAKE), FAKE, k.get("M", 64), k.get("N", 64), 64, nv.BF16, nv.BF16, C.byref(f),
                                                FAKE, 1 << 30, None, None, None, 0)
    assert fw(wq=None) == nv.EINVAL
    assert fw(N=72) == nv.ESHAPE
    assert fw(wq=FAKE + 16) == nv.EALIGN
    bw = nv.lib.nvfp4_linear_bwd_wq(FAKE, FAKE, None, FAKE, FAKE, 64, 64, 64, nv.BF16, nv.BF16, C.byref(f), 0, FAKE, 1 << 30, None, None, None)
    assert bw == nv.EINVAL


def test_swiglu_backward_scalar_step_equals_the_oracle_bit_for_bit():
    # the kernels' own inline function for the SwiGLU backward (compiled for the host) against the oracle's fixed
    # binary32 evaluation: every bit, over gates from deep saturation to deep saturation, zeros and signed zeros
    rng = np.random.default_rng(3)
    n = 200000
    g = np.concatenate([rng.standard_normal(n // 2) * 4.0, rng.uniform(-120.0, 120.0, n // 2 - 8), [0.0, -0.0, 87.0, -87.0, 88.5, -88.5, 1e-30, -1e-30]]).astype(np.float32)
    u = (rng.standard_normal(n) * 1.5).astype(np.float32)
    h = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    dg, du = np.empty(n, np.float32), np.empty(n, np.float32)
    nv.lib.nvfp4_host_swiglu_bwd(_p(h), _p(g), _p(u), n, _p(dg), _p(du))
    og, ou = oracle.swiglu_bwd(h.reshape(1, n), g.reshape(1, n), u.reshape(1, n))
    assert np.array_equal(dg.view(np.uint32), og.reshape(-1).view(np.uint32))
    assert np.array_equal(du.view(np.uint32), ou.reshape(-1).view(np.uint32))


def test_swiglu_and_dyq_argument_errors():
    f = nv.NVFP4.c()
    ops = nv._DualOperands(FAKE, FAKE, FAKE, FAKE, FAKE, 0)
    sq = lambda **k: nv.lib.nvfp4_swiglu_bwd_quantize(k.get("dH", FAKE), FAKE, k.get("U", FAKE), k.get("dt", nv.BF16), k.get("M", 64), k.get("F", 64), 1, 2,
                                                      C.byref(k.get("f", f)), C.byref(k.get("dG", ops)), C.byref(ops), k.get("sg", None), k.get("su", None), k.get("ws", FAKE), k.get("wsb", 1 << 20), None)
    assert sq(dH=None) == nv.EINVAL
    assert sq(sg=FAKE) == nv.EINVAL                      # the two result tensors come together or not at all
    assert sq(sg=FAKE + 4, su=FAKE) == nv.EALIGN
    assert sq(U=None) == nv.EINVAL
    assert sq(dt=4) == nv.EINVAL
    assert sq(M=72) == nv.ESHAPE
    assert sq(F=24) == nv.ESHAPE
    assert sq(f=nv.Format(64, nv.SCALE_E4M3, 1).c()) == nv.EUNSUPPORTED
    assert sq(ws=None) == nv.EWORKSPACE
    assert sq(wsb=100) == nv.EWORKSPACE
    assert sq(dG=nv._DualOperands(FAKE, FAKE, None, FAKE, FAKE, 0)) == nv.EINVAL
    assert sq(dG=nv._DualOperands(FAKE, FAKE, FAKE, FAKE, FAKE, 8)) == nv.EINVAL
    assert sq(dG=nv._DualOperands(FAKE, FAKE, FAKE, FAKE, FAKE, nv.SLAB_ROWS)) == nv.ESHAPE     # F = 64: no whole K tile
    assert sq(dG=nv._DualOperands(FAKE + 8, FAKE, FAKE, FAKE, FAKE, 0)) == nv.EALIGN
    assert nv.lib.nvfp4_swiglu_bwd_workspace_bytes(4096, 11008) >= 4096
    bq = lambda **k: nv.lib.nvfp4_linear_bwd_dyq(k["dy"] if "dy" in k else C.byref(ops), FAKE, FAKE, None, FAKE, FAKE, 64, k.get("N", 64), 64, nv.BF16, nv.BF16,
                                                  C.byref(f), 0, FAKE, 1 << 30, None, None, None)
    assert bq(dy=None) == nv.EINVAL
    assert bq(dy=C.byref(nv._DualOperands(FAKE, FAKE, FAKE, FAKE, None, 0))) == nv.EINVAL
    assert bq(dy=C.byref(nv._DualOperands(None, FAKE, FAKE, FAKE, FAKE, 0))) == nv.EINVAL
    assert bq(dy=C.byref(nv._DualOperands(FAKE, FAKE, FAKE, FAKE, FAKE, nv.SLAB_ROWS))) == nv.EUNSUPPORTED  # the small GEMM takes no slabs
    assert bq(N=72) == nv.ESHAPE


def test_cross_check_switches_round_trip():
    before = nv.cross_check_switches()
    assert 0 <= before <= 7
    assert nv.cross_check_switches(nv.SWITCH_PLAIN_OPERANDS) == before
    assert nv.cross_check_switches() == nv.SWITCH_PLAIN_OPERANDS
    assert nv.cross_check_switches(0xFFFFFFFF) == nv.SWITCH_PLAIN_OPERANDS and nv.cross_check_switches() == 7
    nv.cross_check_switches(before)
    assert nv.cross_check_switches() == before


def test_quantize_dual_argument_errors():
    def dual(x=FAKE, dt=nv.BF16, rows=64, cols=64, ld=64, rnd=nv.SR, fmt=nv.NVFP4, cr=FAKE, sr=FAKE, cc=FAKE,
             sc=FAKE, ts=FAKE, flags=0, ws=FAKE, ws_bytes=1 << 20, k2=nv.SR):
        f = fmt.c()
        return nv.lib.nvfp4_quantize_dual(x, dt, rows, cols, ld, rnd, 1, k2, 2, C.byref(f), cr, sr, cc, sc, ts, flags,
                                          ws, ws_bytes, None)
    assert dual(x=None) == nv.EINVAL
    assert dual(cc=None) == nv.EINVAL
    assert dual(sr=None) == nv.EINVAL
    assert dual(rnd=2) == nv.EINVAL
    assert dual(k2=5) == nv.EINVAL
    assert dual(flags=8) == nv.EINVAL
    # slab outputs: NVFP4 and MXFP4 only, through the one-pass kernel only, whole K tiles of 128 only
    assert dual(flags=nv.SLAB_ROWS) == nv.ESHAPE                      # cols = 64
    assert dual(flags=nv.SLAB_COLS, cols=128, ld=128) == nv.ESHAPE    # rows = 64
    assert dual(flags=nv.SLAB_ROWS, fmt=nv.Format(32, nv.SCALE_E4M3, 1), rows=128, cols=128, ld=128) == nv.EUNSUPPORTED
    assert dual(flags=nv.SLAB_ROWS, rows=128, cols=128, ld=128, rnd=nv.SR, k2=nv.RTN) == nv.EUNSUPPORTED
    assert dual(rows=72) == nv.ESHAPE                     # both axes are blocked
    assert dual(cols=72, ld=72) == nv.ESHAPE
    assert dual(rows=96, cols=96, ld=96, fmt=nv.Format(64, 0, 1)) == nv.ESHAPE
    assert dual(cr=FAKE + 4) == nv.EALIGN
    assert dual(ws=None) == nv.EWORKSPACE
    assert dual(fmt=nv.Format(16, nv.SCALE_E8M0, 1)) == nv.EUNSUPPORTED
    assert dual(rows=0, cr=None, sr=None, cc=None, sc=None, ws=None, fmt=nv.MXFP4) == nv.OK  # empty: nothing launched


def test_gemm_and_linear_argument_errors():
    f = nv.NVFP4.c()
    g = lambda **k: nv.lib.nvfp4_gemm(k.get("M", 64), k.get("N", 64), k.get("K", 64), C.byref(k.get("f", f)),
                                      k.get("a", FAKE), FAKE, FAKE, FAKE, FAKE, k.get("out", FAKE),
                                      k.get("odt", nv.F32), k.get("ldc", 64), None)
    assert g(a=None) == nv.EINVAL
    assert g(odt=9) == nv.EINVAL
    assert g(K=48) == nv.ESHAPE      # multiple of the block but not of 32
    assert g(K=0) == nv.ESHAPE
    assert g(ldc=8) == nv.ESHAPE
    assert g(out=FAKE + 4) == nv.EALIGN
    assert g(f=nv.Format(64, nv.SCALE_E8M0, 0).c()) == nv.EUNSUPPORTED  # E8M0 GEMM exists for block 32 only
    assert g(M=0) == nv.OK           # empty product: nothing to do, nothing launched
    assert g(K=(1 << 23) + 32) == nv.ESHAPE  # contraction length beyond the kernels' 32-bit tile offsets
    # slab operands: only where the large-tile kernel runs (NVFP4, K % 128 == 0, >= 128 tiles of 256 x 256)
    gs = lambda M, N, K, fmt=nv.NVFP4, a=1, b=0: nv.lib.nvfp4_gemm_slab(M, N, K, C.byref(fmt.c()), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE,
                                                                        nv.F32, N, a, b, None)
    assert gs(64, 64, 128) == nv.EUNSUPPORTED
    assert gs(4096, 4096, 192) == nv.EUNSUPPORTED
    assert gs(4096, 4096, 256, nv.MXFP4) == nv.EUNSUPPORTED      # MXFP4: the direct-to-LDS kernel needs K >= 512
    assert gs(4096, 4096, 4096, nv.Format(32, nv.SCALE_E4M3, 1)) == nv.EUNSUPPORTED
    takes = lambda M, N, K, fmt=nv.NVFP4: nv.lib.nvfp4_gemm_takes_slabs(M, N, K, C.byref(fmt.c()))
    assert takes(4096, 11008, 4096) == 1 and takes(2944, 3200, 2816) == 1
    assert takes(2048, 2048, 4096) == 0 and takes(4096, 4096, 4096 + 64) == 0
    assert takes(4096, 4096, 4096, nv.MXFP4) == 1 and takes(64, 64, 512, nv.MXFP4) == 1 and takes(64, 64, 384, nv.MXFP4) == 0
    # slab buffers: rows padded to whole slabs of 256
    assert nv.lib.nvfp4_slab_codes_bytes(256, 128) == 16384 and nv.lib.nvfp4_slab_scales_bytes(256, 128) == 2048
    assert nv.lib.nvfp4_slab_codes_bytes(257, 256) == 2 * 2 * 16384 and nv.lib.nvfp4_slab_scales_bytes(1, 128) == 2048
    assert nv.lib.nvfp4_slab_codes_bytes(0, 128) == 0
    # (MXFP4: 4 scale bytes per row and K tile, half of what the query states)
    assert nv.slab_scales_bytes(257, 256, nv.MXFP4) == 2 * 2 * 1024 and nv.slab_scales_bytes(257, 256) == 2 * 2 * 2048
    fw = lambda **k: nv.lib.nvfp4_linear_fwd(k.get("X", FAKE), FAKE, FAKE, k.get("M", 64), 64, k.get("K", 64), nv.BF16,
                                             nv.F32, C.byref(f), k.get("ws", FAKE), k.get("wsb", 1 << 30), None, None,
                                             k.get("saved"), 0)
    assert fw(X=None) == nv.EINVAL
    assert fw(K=40) == nv.ESHAPE
    assert fw(ws=None) == nv.EWORKSPACE
    assert fw(wsb=16) == nv.EWORKSPACE
    assert fw(M=48, saved=FAKE) == nv.ESHAPE     # X^T is blocked along M for the backward call
    assert fw(saved=FAKE + 16) == nv.EALIGN
    assert nv.linear_saved_bytes(4096, 11008, 4096) >= 4096 * (4096 + 11008) * 9 // 16
    bw = lambda **k: nv.lib.nvfp4_linear_bwd(k.get("dY", FAKE), FAKE, FAKE, FAKE, FAKE, k.get("M", 64), 64, 64,
                                             nv.BF16, nv.F32, C.byref(f), 0, FAKE, k.get("wsb", 1 << 30), None, None,
                                             k.get("saved"))
    assert bw(dY=None) == nv.EINVAL
    assert bw(M=48) == nv.ESHAPE     # the update GEMM contracts over M
    assert bw(wsb=16) == nv.EWORKSPACE
    assert bw(saved=FAKE + 16) == nv.EALIGN


# ---------------------------------------------------------------- scalar steps vs the oracle
def test_host_e4m3_encode_matches_oracle():
    hi = int(np.float32(500.0).view(np.uint32))
    x = np.arange(0, hi, 211, dtype=np.uint32).view(np.float32)
    grid = np.array([oracle.e4m3_decode(b) for b in range(127)], dtype=np.float32)
    mids = ((grid[:-1].astype(np.float64) + grid[1:]) / 2).astype(np.float32)
    sp = np.concatenate([grid, mids])
    sp = np.concatenate([sp, np.nextafter(sp, np.float32(1e9)), np.nextafter(sp, np.float32(-1))])
    x = np.ascontiguousarray(np.concatenate([x, sp[sp >= 0], np.float32([1e4, 3e38])]))
    got = np.empty(x.size, np.uint8)
    nv.lib.nvfp4_host_e4m3_encode_n(_p(x), x.size, _p(got))
    assert np.array_equal(got, oracle.e4m3_encode(x))
    for b in range(127):
        assert nv.lib.nvfp4_host_e4m3_decode(b) == oracle.e4m3_decode(b)


def test_host_round_rtn_matches_oracle_on_every_float_in_range():
    # every binary32 pattern in [2^-3, 6]; below 2^-3 a strided sample (all map to code 0)
    lo, hi = int(np.float32(0.125).view(np.uint32)), int(np.float32(6.0).view(np.uint32))
    for a in range(lo, hi + 1, 1 << 22):
        x = np.arange(a, min(a + (1 << 22), hi + 1), dtype=np.uint32).view(np.float32)
        got = np.empty(x.size, np.uint8)
        nv.lib.nvfp4_host_round_rtn_n(_p(x), x.size, _p(got))
        assert np.array_equal(got, oracle.round_rtn(x))
    x = np.arange(0, lo, 4099, dtype=np.uint32).view(np.float32)
    got = np.empty(x.size, np.uint8)
    nv.lib.nvfp4_host_round_rtn_n(_p(x), x.size, _p(got))
    assert np.array_equal(got, oracle.round_rtn(x)) and got.max() == 0


def test_host_round_sr_matches_oracle():
    rng = np.random.default_rng(0)
    hi = int(np.float32(6.0).view(np.uint32))
    # random magnitudes x random draws, plus every draw for magnitudes around each threshold
    m = rng.integers(0, hi + 1, 4_000_000, dtype=np.uint32).view(np.float32)
    u = rng.integers(0, 65536, m.size, dtype=np.uint32)
    got = np.empty(m.size, np.uint8)
    nv.lib.nvfp4_host_round_sr_n(_p(m), _p(u), m.size, _p(got))
    assert np.array_equal(got, oracle.round_sr(m, u))
    uu = np.arange(65536, dtype=np.uint32)
    for mv in [0.0, 1e-30, 0.1, 0.25, 0.4999999, 0.5, 0.75, 1.0, 1.2, 1.9999999, 2.0, 2.4, 3.0, 3.999999, 4.0, 5.0,
               5.9999995, 6.0, 2.0 ** -17 * 0.5, 0.5 + 2.0 ** -18, 4 + 2.0 ** -16,
               # exact ties between the position and a centred draw, one per binade of the grid
               0.5 * 100.5 / 65536, 0.5 + 0.5 * 7.5 / 65536, 1.5 + 0.5 * 65535.5 / 65536, 2 + 100.5 / 65536,
               3 + 0.5 / 65536, 4 + 2 * 32767.5 / 65536]:
        mm = np.full(65536, mv, np.float32)
        nv.lib.nvfp4_host_round_sr_n(_p(mm), _p(uu), 65536, _p(got[:65536]))
        assert np.array_equal(got[:65536], oracle.round_sr(mm, uu)), mv


def test_host_philox_and_sr_bits(golden_dir):
    for ln in open(os.path.join(golden_dir, "philox4x32_10_kat.txt")):
        if ln.startswith("#") or not ln.strip():
            continue
        w = [int(t, 16) for t in ln.split()]
        c, k, out = np.array(w[0:4], np.uint32), np.array(w[4:6], np.uint32), np.empty(4, np.uint32)
        nv.lib.nvfp4_host_philox4x32_10(_p(c), _p(k), _p(out))
        assert [int(v) for v in out] == w[6:10]
    seed = 0xFEDCBA9876543210
    for e0 in (0, 8 * 12345, (1 << 36) + 24):
        want = oracle.sr_bits_range(seed, e0, 64)
        assert [nv.lib.nvfp4_host_sr_bits(seed, e0 + t) for t in range(64)] == [int(v) for v in want]


def test_host_e8m0_matches_oracle_rule():
    rng = np.random.default_rng(1)
    a = np.abs(rng.standard_normal(2000).astype(np.float32)) * np.float32(10) ** rng.integers(-30, 30, 2000).astype(np.float32)
    a = np.concatenate([a, np.float32([1e-45, 1e-40, 2.0 ** -126, 2.0 ** -127, 1.0, 6.0, 7.99, 8.0, 3e38])]).astype(np.float32)
    for v in a:
        x = np.zeros((1, 32), np.float32)
        x[0, 0] = v
        want = oracle.quantize(x, 1, oracle.RTN, 0, oracle.MXFP4)[1][0, 0]
        assert nv.lib.nvfp4_host_e8m0_encode(float(v)) == want, v


def test_gemm_tile_rule():
    E4, MX = nv.NVFP4, nv.MXFP4
    assert nv.gemm_tile(0, 64, 64, E4) == (0, 0) and nv.gemm_tile(64, 64, 64, nv.Format(8, 0, 1)) == (0, 0)
    # MXFP4 contractions shorter than a K tile have the large tiles too (on 64 x 64, 4096 x 11008 x 64 took 82 us, on 128 x 128 20)
    for K in (32, 64, 96):
        assert nv.gemm_tile(4096, 11008, K, MX) == (128, 128)
    # short contractions with E4M3 scales: 128 x 256 tiles only pay where the products fill the time between their epilogues
    # (8192 x 8192 x 256, bf16 outputs: 45.6 us on 128 x 128, 55 on the larger ones)
    for M, N, K in ((8192, 8192, 128), (8192, 8192, 256), (4096, 11008, 128), (4096, 11008, 256), (8192, 4096, 256)):
        assert nv.gemm_tile(M, N, K, E4) == (128, 128)
    # MXFP4, 256 tiles of 256 x 128: one per CU, no faster than 256 x 256 and slower than 128 x 128
    assert nv.gemm_tile(2048, 4096, 4096, MX) == (128, 128) and nv.gemm_tile(2048, 4096, 11008, MX) == (128, 128)


def test_four_group_tiles_take_one_round():
    four = lambda M, N, K: nv.gemm_split(M, N, K, nv.NVFP4) == 4 and nv.gemm_tile(M, N, K, nv.NVFP4) in ((96, 128), (128, 128))
    for M, N, K in ((1056, 2080, 2784), (1536, 1536, 6144), (1376, 2432, 12032), (704, 4832, 4992), (192, 11424, 2432)):
        assert four(M, N, K), (M, N, K)
    # with more than one workgroup per CU they were slower than the tile without groups by as much as 23 %
    for M, N, K in ((3072, 1792, 8256), (2377, 1793, 7552), (1968, 2752, 6720), (1280, 6816, 5760), (1381, 5979, 8800), (2400, 3680, 11392),
                    (672, 11008, 4096), (3355, 5317, 10016)):
        assert not four(M, N, K), (M, N, K)
    assert nv.gemm_split(16, 4096, 4096) == 8 and nv.gemm_split(4096, 4096, 4096) == 1 and nv.gemm_split(0, 1, 1) == 0


def test_which_quantizers_stream():
    # (rows, cols, rounding of rows or None, of columns, format, preset): slower in the walk of resident workgroups, by 4 to 46 %, or faster
    RTN, SR, E64, E128, X16 = nv.RTN, nv.SR, nv.Format(64, 0, 1), nv.Format(128, 0, 1), nv.Format(16, 1, 0)
    X64 = nv.Format(64, 1, 0)
    slower = [(14528, 10168, None, RTN, E64, 1), (14784, 7544, None, RTN, E64, 0), (12608, 11016, None, RTN, X64, 0), (8704, 16896, None, RTN, E128, 1),
              (10560, 10232, None, SR, E64, 1), (26432, 6104, None, SR, E64, 1), (16896, 8576, None, SR, E128, 1), (12608, 9760, None, SR, nv.MXFP4, 0),
              (16896, 9216, None, RTN, nv.MXFP4, 0), (3904, 6912, None, RTN, nv.MXFP4, 0), (5376, 5992, None, RTN, nv.NVFP4, 1), (18432, 7168, None, RTN, nv.NVFP4, 1),
              (36672, 4016, None, RTN, X16, 0), (9664, 6640, None, SR, E64, 1), (14656, 10600, None, SR, E64, 0), (2752, 23528, None, SR, X64, 0), (6400, 3456, RTN, RTN, X16, 0), (4224, 7552, RTN, RTN, nv.MXFP4, 0), (6912, 2560, RTN, RTN, nv.MXFP4, 0), (5632, 4736, RTN, RTN, nv.NVFP4, 1)]
    faster = [(4096, 11008, None, RTN, nv.NVFP4, 0), (4096, 11008, None, RTN, nv.MXFP4, 0), (8192, 12288, None, RTN, nv.NVFP4, 0), (8192, 8192, None, SR, nv.NVFP4, 0),
              (8192, 8192, None, SR, nv.NVFP4, 1), (8192, 8192, None, SR, nv.MXFP4, 0), (4096, 8192, None, SR, E64, 1), (16384, 8192, None, SR, E128, 0),
              (4096, 11008, RTN, RTN, nv.MXFP4, 0), (4096, 8192, RTN, SR, nv.MXFP4, 0), (8192, 8192, SR, SR, nv.MXFP4, 0), (3072, 6144, RTN, RTN, nv.NVFP4, 1)]
    for calls, want in ((slower, False), (faster, True)):
        for rows, cols, rr, rc, fmt, preset in calls:
            assert nv.quantize_streams(rows, cols, cols, rr is not None, rr or 0, rc, fmt, nv.PRESET_TSCALE if preset else 0) == want, (rows, cols, rr, rc, fmt, preset)
    # small tensors, many tiles or not; a row pitch beyond 32-bit offsets; ragged rows of columns
    assert not nv.quantize_streams(131072, 32, 32, False, 0, RTN) and not nv.quantize_streams(8192, 8192, (1 << 22) + 8, False, 0, SR)
    assert not nv.quantize_streams(8192, 8196, 8200, False, 0, SR) and not nv.quantize_streams(8192, 8192, 8192, True, SR, RTN)
    assert nv.quantize_streams(16384, 12288, 12288, True, RTN, RTN, nv.MXFP4, nv.SLAB_ROWS | nv.SLAB_COLS)
    assert not nv.quantize_streams(5120, 5120, 5120, True, RTN, RTN, nv.MXFP4, nv.SLAB_ROWS | nv.SLAB_COLS)


def test_fused_layers_by_workgroups():
    # the workgroups of a fused layer repeat each other's quantization, so what counts is their number, not the tensors' bytes alone (1024 x
    # 1024 x 64, forward, 28 us in one launch of 1024, 10 in two): (forward, with saved operands, backward on these)
    import torch
    bf16, f32, U = torch.bfloat16, torch.float32, nv.Format(16, 0, 0)
    for shape, dtype, fmt, want in (
            ((64, 256, 128), f32, nv.NVFP4, (True, True, True)), ((32, 32, 32), bf16, nv.MXFP4, (True, True, True)),
            ((480, 512, 64), bf16, nv.NVFP4, (True, True, False)), ((512, 512, 64), bf16, nv.NVFP4, (True, False, False)),
            ((512, 544, 64), bf16, nv.NVFP4, (False, False, False)), ((512, 512, 64), f32, nv.NVFP4, (True, True, False)),
            ((1024, 512, 32), f32, nv.NVFP4, (True, False, False)), ((1024, 544, 32), f32, nv.NVFP4, (False, False, False)),
            ((128, 128, 256), bf16, nv.NVFP4, (True, True, True)), ((128, 128, 288), bf16, nv.NVFP4, (False, True, True)), ((128, 128, 512), bf16, U, (True, True, True)),
            ((1024, 768, 64), bf16, nv.MXFP4, (True, True, False)), ((1024, 800, 64), bf16, nv.MXFP4, (False, True, False)),
            ((1024, 992, 64), bf16, nv.MXFP4, (False, False, False)), ((1024, 512, 32), bf16, U, (True, True, False)), ((1024, 544, 32), bf16, U, (False, False, False)),
            ((256, 256, 672), bf16, nv.NVFP4, (False, False, True)), ((256, 256, 704), bf16, nv.NVFP4, (False, False, False)), ((256, 256, 4096), bf16, nv.MXFP4, (False, False, False)),
            ((128, 128, 1344), bf16, nv.NVFP4, (False, False, True)), ((128, 128, 1376), bf16, nv.NVFP4, (False, False, False)), ((128, 128, 8192), bf16, nv.NVFP4, (False, False, False)),
            ((64, 512, 832), bf16, nv.NVFP4, (False, False, False)), ((64, 512, 832), f32, nv.NVFP4, (False, False, True)), ((64, 64, 2880), f32, nv.NVFP4, (False, False, False)),
            ((64, 512, 832), bf16, U, (False, False, True)), ((128, 128, 2720), bf16, nv.MXFP4, (False, False, True)), ((128, 128, 2752), bf16, nv.MXFP4, (False, False, False))):
        assert nv.layer_fused(*shape, dtype, fmt) == want, (shape, dtype, fmt)
    # other blocks, a size of zero
    assert nv.layer_fused(64, 256, 128, f32, nv.Format(32, 0, 1)) == (False, False, False) and nv.layer_fused(0, 32, 32) == (False, False, False)


def test_few_rows_up_to_the_launch_limit():
    # 512 threads for 64 columns, counted in 32 bits: a wider product stays on a tile that can be launched
    last = 64 * ((1 << 32) // 512 - 1)
    assert nv.gemm_few_rows(16, last, 512) and not nv.gemm_few_rows(16, last + 1, 512) and not nv.gemm_few_rows(1, 1 << 29, 512)
    assert nv.gemm_tile(16, 1 << 29, 512) == (64, 64) and ((1 << 29) // 64) * 256 < 1 << 32
    assert nv.gemm_few_rows(16, 16384, 32) and not nv.gemm_few_rows(16, 16385, 480) and nv.gemm_few_rows(16, 16385, 512)
    assert nv.gemm_few_rows(16, 16384, 8192, nv.MXFP4) and not nv.gemm_few_rows(16, 16385, 8192, nv.MXFP4)
    assert not nv.gemm_few_rows(17, 4096, 4096) and not nv.gemm_few_rows(16, 4096, 4096, nv.Format(64, 0, 1)) and not nv.gemm_few_rows(0, 64, 64)


def test_no_tile_beyond_the_launch_limit():
    # a launch counts its threads in 32 bits, and no product that one of the tiles can serve may be given one that cannot
    # (rows, columns, parts of the contraction -> threads)
    threads = {(32, 32, 8): 512, (32, 64, 8): 512, (64, 32, 8): 512, (64, 64, 4): 256, (96, 128, 4): 512, (128, 128, 1): 256, (128, 128, 4): 512,
               (128, 256, 1): 512, (128, 256, 2): 512, (160, 256, 1): 512, (192, 256, 1): 512, (256, 128, 1): 256, (256, 256, 1): 512}
    seen = set()
    for fmt in (nv.NVFP4, nv.MXFP4):
        for M in (1, 64, 300, 2700, 2970, 4096, 1 << 18, 1 << 20, 1 << 24, 1 << 26, 1 << 28, (1 << 28) + 1, 1 << 30):
            for N in (1, 32, 33, 64, 128, 300, 641, 1093, 4096, 1 << 18):
                for K in (32, 96, 128, 512, 1024, 1536, 2560, 4096, 16384):
                    if M * N > 1 << 38:  # (more than 256 x 256 tiles can serve)
                        continue
                    t = nv.gemm_tile(M, N, K, fmt) + (nv.gemm_split(M, N, K, fmt),)
                    seen.add(t)
                    assert -(-M // t[0]) * -(-N // t[1]) * threads[t] < 1 << 32, (M, N, K, t)
    assert {(96, 128, 4), (128, 128, 4), (128, 128, 1), (256, 256, 1)} <= seen


def test_formats_keep_nothing_of_a_call():
    # what c() returns is the caller's to change; a format's own fields are all that it holds, copied, pickled and unpacked as such
    import copy
    import pickle
    for fmt in (nv.NVFP4, nv.MXFP4, nv.Format(64, nv.SCALE_E4M3, 1)):
        fields = dict(block=fmt.block, scale=fmt.scale, tensor_scale=fmt.tensor_scale)
        c = fmt.c()
        c.block, c.scale, c.tensor_scale = 7, 8, 9
        again = fmt.c()
        assert (again.block, again.scale, again.tensor_scale) == tuple(fields.values())
        assert vars(fmt) == fields and nv.Format(**vars(fmt)) == fmt and copy.deepcopy(fmt) == pickle.loads(pickle.dumps(fmt)) == fmt
    with pytest.raises(TypeError):
        nv.Format(16.0, nv.SCALE_E4M3, 1).c()


def test_known_sizes():
    # by value, of both calls and all formats, and not without bound
    for M in range(32, 32 * 1200, 32):
        for name in ("nvfp4_linear_fwd_workspace_bytes", "nvfp4_linear_bwd_workspace_bytes"):
            f = (nv.NVFP4 if M % 64 else nv.MXFP4).c()
            assert nv._workspace_bytes(name, M, 64, 96, f) == getattr(nv.lib, name)(M, 64, 96, C.byref(f))
    assert len(nv._known_sizes) <= 1000
    assert nv._workspace_bytes("nvfp4_linear_fwd_workspace_bytes", 64, 96, 128, nv.Format(7, 8, 9).c()) == 0  # (a format that the library refuses)


@pytest.mark.parametrize("lacking", [None, "_raw_alloc", "_raw_delete", "_raw_device"])
def test_a_block_that_could_not_be_had(lacking, monkeypatch):
    # out of memory, with and without torch's raw entries: the caller gets that error, and nothing else is reported about the half-made block
    import gc
    import sys

    def no_memory(*a, **k):
        raise MemoryError("no memory")

    like = type("Tensor", (), {"get_device": lambda self: 0, "device": "cpu"})()
    unraisable, freed = [], []
    monkeypatch.setattr(sys, "unraisablehook", lambda u: unraisable.append(u.exc_value))
    monkeypatch.setattr(nv, "_raw_device", lambda: 0)
    monkeypatch.setattr(nv, "_raw_alloc", no_memory)
    monkeypatch.setattr(nv, "_raw_delete", freed.append)
    monkeypatch.setattr(nv.torch, "empty", no_memory)
    if lacking:
        monkeypatch.setattr(nv, lacking, None)
    with pytest.raises(MemoryError):
        nv._Block(64, like, 0)
    gc.collect()
    assert not unraisable and not freed


def test_two_group_tiles_are_of_long_contractions():
    # 128 x 256 in two groups has a kernel for contractions of more than seven K tiles only, and the rule names it for those only
    for K in range(32, 7 * 128 + 1, 32):
        for M in list(range(128, 8193, 384)) + [2048]:
            for N in list(range(256, 12289, 768)) + [4096]:
                assert nv.gemm_split(M, N, K) == 1 or nv.gemm_tile(M, N, K) != (128, 256), (M, N, K)
    for M, N, K in ((2048, 4096, 1536), (2048, 4096, 4096), (8204, 580, 1472)):
        assert nv.gemm_tile(M, N, K) == (128, 256) and nv.gemm_split(M, N, K) == 2
