"""The GEMM at the sizes where its tiles can go wrong: every workgroup tile the size rule chooses from, with whole and ragged
contractions (one K tile, less than one, one more than the waves that share it), rows and columns past the edge, one-row and
one-column outputs.  Against the fp64 oracle, completely where it is cheap, on sampled outputs otherwise."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_bf16_gemm_close, assert_gemm_close, ofmt, to_np

pytestmark = pytest.mark.gpu

nv = None


@pytest.fixture(scope="module", autouse=True)
def _binding():
    global nv
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2505_19115_amd import binding
    nv = binding
    yield


FORMATS = {"nvfp4": (16, 0), "e4m3_32": (32, 0), "e4m3_64": (64, 0), "e4m3_128": (128, 0), "mxfp4": (32, 1)}


def operand(rng, rows, K, block, scale):
    codes = rng.integers(0, 256, (rows, K // 2)).astype(np.uint8)
    lo, hi = (118, 136) if scale else (0x01, 0x7F)  # (every finite E4M3 byte; E8M0 exponents within 2^9)
    return codes, rng.integers(lo, hi, (rows, K // block)).astype(np.uint8), 1.0 if scale else 0.75


def run(A, B, fmt, out_dtype):
    dev = lambda o: (torch.from_numpy(o[0]).cuda(), torch.from_numpy(o[1]).cuda(), torch.tensor([o[2]], dtype=torch.float32, device="cuda"))
    Y = nv.gemm(dev(A), dev(B), fmt, out_dtype)
    torch.cuda.synchronize()
    return to_np(Y.float())


def close(got, ref, ref_abs, what, out_dtype):
    (assert_bf16_gemm_close if out_dtype == torch.bfloat16 else assert_gemm_close)(got, ref, ref_abs, what)


@pytest.mark.parametrize("fmt_name", FORMATS)
@pytest.mark.parametrize("shape", [(1, 1, 32), (31, 33, 64), (33, 65, 96), (64, 64, 128), (65, 31, 160), (128, 129, 384),
                                   (2, 96, 1024), (16, 200, 1152), (70, 300, 2208), (1, 257, 4128)])
def test_small_products(shape, fmt_name):
    block, scale = FORMATS[fmt_name]
    M, N, K = shape
    K = -(-K // max(block, 32)) * max(block, 32)
    fmt = nv.Format(block, scale, 1 - scale)
    out_dtype = torch.float32 if (M + N) % 2 == 0 else torch.bfloat16
    rng = np.random.default_rng(M + 7 * N + K)
    A, B = operand(rng, M, K, block, scale), operand(rng, N, K, block, scale)
    print(f"[case] gemm tile {fmt_name} {M}x{N}x{K} {out_dtype}", flush=True)
    got = run(A, B, fmt, out_dtype)
    of = ofmt(fmt)
    close(got, oracle.gemm_nt(A, B, of), oracle.gemm_nt(A, B, of, take_abs=True), f"{fmt_name} {shape}", out_dtype)


# The tile each shape gets from the size rule, E4M3 and E8M0 scales: asserted, so that a change of the rule moves no test in silence.
# Between them: every tile of both kinds, each with whole K tiles and with a K tail, rows and columns past the edge.
SAMPLED = [((71, 4160, 32), (32, 64), (32, 64)), ((65, 4171, 1152), (32, 64), (32, 64)),
           ((65, 3036, 32), (64, 32), (64, 32)), ((300, 1100, 544), (64, 32), (64, 32)), ((100, 3000, 1024), (64, 32), (64, 32)),
           ((171, 2818, 32), (64, 64), (64, 64)), ((1200, 905, 640), (32, 32), (128, 128)), ((241, 268, 32), (32, 32), (32, 32)),
           ((257, 3401, 160), (128, 128), (128, 128)), ((2081, 1100, 256), (128, 128), (128, 128)),
           ((3666, 1043, 1696), (64, 64), (128, 128)), ((3596, 1033, 1792), (64, 64), (128, 128)),
           ((8195, 1802, 160), None, (256, 128)), ((7171, 2050, 256), None, (256, 128)),
           ((2721, 1418, 128), (128, 256), (128, 128)), ((1618, 3033, 160), (128, 256), (128, 128)),
           ((2505, 3212, 256), (192, 256), (128, 128)), ((2373, 3777, 160), (192, 256), (128, 128)),
           ((2841, 4235, 160), (192, 256), (256, 256)),
           # 256 x 256; in E8M0 the direct-to-LDS kernel takes K = 640 and 1024, the tile kernel the others
           ((2720, 4358, 32), (256, 256), (256, 256)), ((3900, 4080, 160), (256, 256), (256, 256)), ((2709, 4364, 128), (256, 256), (256, 256)),
           ((4030, 4050, 384), (256, 256), (256, 256)), ((3900, 4090, 640), (256, 256), (256, 256)), ((3900, 4080, 1024), (256, 256), (256, 256))]


@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4", "e4m3_32"])
@pytest.mark.parametrize("shape,e4m3_tile,e8m0_tile", SAMPLED, ids=["x".join(map(str, c[0])) for c in SAMPLED])
def test_every_tile_sampled(shape, e4m3_tile, e8m0_tile, fmt_name):
    block, scale = FORMATS[fmt_name]
    M, N, K = shape
    fmt = nv.Format(block, scale, 1 - scale)
    want = e8m0_tile if scale else e4m3_tile
    assert want is None or nv.gemm_tile(M, N, K, fmt) == want
    check_sampled(shape, fmt_name, torch.float32 if K % 256 else torch.bfloat16)


def check_sampled(shape, fmt_name, out_dtype):
    block, scale = FORMATS[fmt_name]
    M, N, K = shape
    fmt = nv.Format(block, scale, 1 - scale)
    rng = np.random.default_rng(M + 7 * N + K)
    A, B = operand(rng, M, K, block, scale), operand(rng, N, K, block, scale)
    print(f"[case] gemm tile sampled {fmt_name} {M}x{N}x{K} {out_dtype}", flush=True)
    got = run(A, B, fmt, out_dtype)
    # random outputs, the first and last rows and columns, and the two rows and columns at every multiple of 32 of a band
    edge = lambda n: np.unique(np.clip(np.concatenate([[0, n - 1, n - 2], np.arange(31, min(n, 520), 32), np.arange(32, min(n, 520), 32)]), 0, n - 1))
    ii = np.concatenate([rng.integers(0, M, 2000), np.repeat(edge(M), 40), rng.integers(0, M, 40 * len(edge(N)))])
    jj = np.concatenate([rng.integers(0, N, 2000), rng.integers(0, N, 40 * len(edge(M))), np.repeat(edge(N), 40)])
    of = ofmt(fmt)
    close(got[ii, jj], oracle.gemm_nt_sample(A, B, ii, jj, of), oracle.gemm_nt_sample(A, B, ii, jj, of, take_abs=True),
          f"{fmt_name} {shape}", out_dtype)
    assert np.isfinite(got).all()


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
def test_window_of_a_wider_output(fmt_name, out_dtype):
    # an odd leading dimension rules wide stores out, one of 4 mod 8 leaves pieces of 8 bytes (bf16); columns beside the window stay untouched
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    rng = np.random.default_rng(5)
    for M, N, K, ld in ((40, 70, 160, 73), (40, 72, 256, 80), (40, 75, 160, 76), (600, 610, 160, 611), (600, 610, 160, 612)):
        A, B = operand(rng, M, K, block, scale), operand(rng, N, K, block, scale)
        dev = lambda o: (torch.from_numpy(o[0]).cuda(), torch.from_numpy(o[1]).cuda(), torch.tensor([o[2]], dtype=torch.float32, device="cuda"))
        print(f"[case] gemm window {fmt_name} {M}x{N}x{K} ldc={ld} {out_dtype}", flush=True)
        out = torch.full((M, ld), -1.0, device="cuda", dtype=out_dtype)
        nv.gemm(dev(A), dev(B), fmt, out=out[:, :N])
        torch.cuda.synchronize()
        of = ofmt(fmt)
        close(to_np(out[:, :N].float()), oracle.gemm_nt(A, B, of), oracle.gemm_nt(A, B, of, take_abs=True), f"ldc {ld}", out_dtype)
        assert bool((out[:, N:] == -1.0).all())


# (a 192-row tile that starts in the middle of a slab reads the end of it and the beginning of the next)
@pytest.mark.parametrize("shape", [pytest.param((2832, 3072, 256), id="192x256"), pytest.param((2352, 3200, 256), id="128x256")])
def test_tiles_across_slabs(shape):
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W = (torch.randn((n, K), generator=g, device="cuda") for n in (M, N))
    print(f"[case] gemm tiles across slabs {M}x{N}x{K}", flush=True)
    plain = nv.gemm(nv.quantize_dual(X)[0], nv.quantize_dual(W)[0], out_dtype=torch.float32)
    for slabs in ((True, False), (False, True), (True, True)):
        A, B = (nv.quantize_dual(t, slab_rows=s)[0] for t, s in ((X, slabs[0]), (W, slabs[1])))
        assert torch.equal(nv.gemm(A, B, out_dtype=torch.float32, slabs=slabs, shape=shape), plain)


# A backward call that wants both gradients runs two small products in one launch, up to 256 workgroups in all (on that line,
# one past it, and one tile each), with the same bits as the two products by themselves.
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("shape", [(32, 32, 32), (64, 256, 128), (96, 160, 1024), (64, 224, 896), (64, 224, 928)])
def test_both_gradients_in_one_launch(shape, fmt_name):
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    X, W, dY = (torch.randn(s, generator=g, device="cuda") for s in ((M, K), (N, K), (M, N)))
    print(f"[case] gradients in one launch {fmt_name} {shape}", flush=True)
    dX, dW = nv.linear_bwd(dY, X, W, 3, fmt)
    assert torch.equal(dX, nv.gemm(nv.quantize(dY, 1, nv.SR, 3, fmt), nv.quantize(W, 0, nv.RTN, 0, fmt), fmt))
    assert torch.equal(dW, nv.gemm(nv.quantize(dY, 0, nv.SR, 4, fmt), nv.quantize(X, 0, nv.SR, 5, fmt), fmt))


# The large kernels' outputs with every kind of row: 16-byte aligned ones with a gap (ldc), ones that start at multiples of 8 bytes
# (bf16, ldc = 4 mod 8) and of one element, at the edges of the output and inside.
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("shape,e4m3_tile,e8m0_tile", [((3900, 4090, 640), (256, 256), (256, 256)), ((4030, 4050, 384), (256, 256), (256, 256)),
                                                       ((2505, 3212, 256), (192, 256), (128, 128)), ((2081, 1100, 256), (128, 128), (128, 128))])
def test_large_tiles_in_windows_of_wider_outputs(shape, e4m3_tile, e8m0_tile, fmt_name, out_dtype):
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    M, N, K = shape
    assert nv.gemm_tile(M, N, K, fmt) == (e8m0_tile if scale else e4m3_tile)
    rng = np.random.default_rng(M)
    A, B = operand(rng, M, K, block, scale), operand(rng, N, K, block, scale)
    dev = lambda o: (torch.from_numpy(o[0]).cuda(), torch.from_numpy(o[1]).cuda(), torch.tensor([o[2]], dtype=torch.float32, device="cuda"))
    a, b = dev(A), dev(B)
    ii, jj = rng.integers(0, M, 3000), rng.integers(0, N, 3000)
    ii[:1500], jj[1000:2500] = rng.integers(M - 260, M, 1500), rng.integers(N - 260, N, 1500)
    of = ofmt(fmt)
    ref, ref_abs = oracle.gemm_nt_sample(A, B, ii, jj, of), oracle.gemm_nt_sample(A, B, ii, jj, of, take_abs=True)
    first = None
    for ld in (-(-N // 8) * 8 + 8, -(-N // 8) * 8 + 4, (N | 1) + 2):
        print(f"[case] gemm windows {fmt_name} {M}x{N}x{K} ldc={ld} {out_dtype}", flush=True)
        out = torch.full((M, ld), -1.0, device="cuda", dtype=out_dtype)
        nv.gemm(a, b, fmt, out=out[:, :N])
        torch.cuda.synchronize()
        got = out[:, :N].float()
        assert bool((out[:, N:] == -1.0).all()), "columns outside the window were written"
        if first is None:
            first = got
            close(to_np(got)[ii, jj], ref, ref_abs, f"ldc {ld}", out_dtype)
        assert torch.equal(got, first)


# MXFP4 contractions shorter than one K tile, on the large tiles
@pytest.mark.parametrize("K", [32, 64, 96])
@pytest.mark.parametrize("shape,tile", [((2052, 1990), (128, 128)), ((2720, 4358), (256, 256))])
def test_mxfp4_short_contractions(shape, tile, K):
    M, N = shape
    assert nv.gemm_tile(M, N, K, nv.MXFP4) == tile
    rng = np.random.default_rng(M + K)
    A, B = operand(rng, M, K, 32, 1), operand(rng, N, K, 32, 1)
    print(f"[case] short contraction {M}x{N}x{K}", flush=True)
    got = run(A, B, nv.MXFP4, torch.float32)
    of = ofmt(nv.MXFP4)
    close(got, oracle.gemm_nt(A, B, of), oracle.gemm_nt(A, B, of, take_abs=True), f"K {K}", torch.float32)


# Operands in slabs on tiles other than the 256 x 256 they were made for: the same bits as row-major operands.  (16 rows: on the kernel for few
# rows, whatever the rule of the tiles answers.)
@pytest.mark.parametrize("fmt_name,shape,tile", [("nvfp4", (16, 32768, 1024), (32, 32)), ("nvfp4", (17, 32768, 1024), (32, 32)), ("nvfp4", (20, 32768, 4096), (32, 64)),
                                                 ("nvfp4", (50, 32800, 1024), (64, 64)),
                                                 ("nvfp4", (96, 32700, 2048), (96, 128)), ("nvfp4", (128, 32768, 4096), (128, 128)),
                                                 ("mxfp4", (40, 2080, 1024), (32, 32)), ("mxfp4", (70, 4100, 1024), (32, 64)),
                                                 ("mxfp4", (100, 3000, 1024), (64, 32)), ("mxfp4", (33, 8200, 512), (64, 64)),
                                                 ("mxfp4", (2048, 4096, 1024), (128, 128)), ("mxfp4", (7171, 2050, 512), (256, 128)),
                                                 ("mxfp4", (3900, 4080, 640), (256, 256))])
def test_slab_operands_on_every_tile(fmt_name, shape, tile):
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    M, N, K = shape
    assert nv.gemm_tile(M, N, K, fmt) == tile and (fmt_name == "mxfp4" or nv.gemm_split(M, N, K, fmt) > 1)
    assert nv.gemm_few_rows(M, N, K, fmt) == (M == 16)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    # (rows padded to whole blocks for the quantizer; the product takes the first M and N of them)
    X, W = (torch.randn((-(-n // block) * block, K), generator=g, device="cuda") for n in (M, N))
    ops = [(nv.quantize_dual(t, fmt=fmt)[0], nv.quantize_dual(t, fmt=fmt, slab_rows=True)[0]) for t in (X, W)]
    print(f"[case] slabs {fmt_name} {M}x{N}x{K}", flush=True)
    plain = nv.gemm(ops[0][0], ops[1][0], fmt, shape=shape)
    for slabs in ((True, False), (False, True), (True, True)):
        assert torch.equal(nv.gemm(ops[0][slabs[0]], ops[1][slabs[1]], fmt, slabs=slabs, shape=shape), plain), slabs


@pytest.mark.parametrize("M", [16, 24])
def test_packed_weights_of_a_wide_projection(M):
    # few tokens against a vocabulary-sized weight: its packed operand is in slabs (128 output tiles of 256 x 256), the product runs on
    # the kernel for few rows or on a tile whose waves divide the contraction
    N, K = 32768, 512
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X, W = (torch.randn((n, K), generator=g, device="cuda").to(torch.bfloat16) for n in (M, N))
    assert nv.gemm_tile(M, N, K)[0] <= 64 and nv.lib.nvfp4_gemm_takes_slabs(M, N, K, ctypes.byref(nv.NVFP4.c()))
    assert nv.gemm_few_rows(M, N, K) == (M == 16)
    Y = nv.linear_fwd(X, None, w_operands=nv.quantize_weight(W, M), N=N)
    assert torch.equal(Y, nv.linear_fwd(X, W))
    assert torch.equal(Y, nv.gemm(nv.quantize(X), nv.quantize(W)))


# Tiles whose four groups of waves take every fourth K tile: every remainder of the K tiles (the groups without a K tile in the last step
# add zeros), with whole K tiles and with a K tail, rows and columns past the edge, both output types.
FOUR_GROUPS = [((2970, 641, 1536), (96, 128)), ((1667, 1175, 1472), (96, 128)), ((2970, 642, 2176), (96, 128)), ((1798, 1098, 2112), (96, 128)),
               ((708, 2692, 1792), (96, 128)), ((716, 2689, 1728), (96, 128)), ((2955, 648, 1408), (96, 128)), ((646, 2971, 1344), (96, 128)),
               ((3081, 963, 2560), (128, 128)), ((1106, 2689, 2496), (128, 128)), ((1222, 2442, 5248), (128, 128)), ((2890, 1028, 5184), (128, 128)),
               ((2232, 1351, 4352), (128, 128)), ((1930, 1553, 4288), (128, 128)), ((1094, 2713, 3456), (128, 128)), ((1094, 2760, 3392), (128, 128))]


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "e4m3_64"])
@pytest.mark.parametrize("shape,tile", FOUR_GROUPS, ids=["x".join(map(str, c[0])) for c in FOUR_GROUPS])
def test_four_groups_sampled(shape, tile, fmt_name, out_dtype):
    assert nv.gemm_tile(*shape) == tile and nv.gemm_split(*shape) == 4
    check_sampled(shape, fmt_name, out_dtype)


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["e4m3_32", "e4m3_128"])
@pytest.mark.parametrize("shape,tile", [((2955, 648, 1408), (96, 128)), ((1094, 2713, 3456), (128, 128))])
def test_four_groups_of_other_blocks(shape, tile, fmt_name, out_dtype):
    assert nv.gemm_tile(*shape) == tile and nv.gemm_split(*shape) == 4
    check_sampled(shape, fmt_name, out_dtype)


# Row-major scales are fetched 8 bytes of a row at a time, the last 8 ending with the row: rows of fewer than 8 bytes, of 8, of one more,
# of whole windows and one K tile past them, at every block size.
@pytest.mark.parametrize("fmt_name,K", [("nvfp4", 32), ("nvfp4", 96), ("nvfp4", 160), ("nvfp4", 288), ("e4m3_32", 32), ("e4m3_32", 224),
                                        ("e4m3_32", 256), ("e4m3_32", 288), ("e4m3_32", 640), ("e4m3_64", 64), ("e4m3_64", 448),
                                        ("e4m3_64", 512), ("e4m3_64", 576), ("e4m3_64", 1152), ("e4m3_128", 128), ("e4m3_128", 896),
                                        ("e4m3_128", 1024), ("e4m3_128", 1152), ("e4m3_128", 2176)])
@pytest.mark.parametrize("M,N,tile", [(2720, 4358, (256, 256)), (1056, 2080, None)])
def test_windows_of_row_major_scales(M, N, tile, fmt_name, K):
    assert nv.gemm_tile(M, N, K) == (tile or ((128, 128) if K < 2176 else (96, 128)))
    check_sampled((M, N, K), fmt_name, torch.float32)


# Packed weights of more than a few million elements are slabs also where few tokens meet them: every tile of up to 64 x 64 and both with
# four groups, the other operand row-major, output columns that end inside a slab; the bits of the calls that quantize W themselves.
FEW_TOKENS = [((32, 2080, 2176), (32, 32), 8), ((160, 2080, 2176), (64, 32), 8), ((224, 2080, 2176), (32, 64), 8), ((320, 2080, 2176), (64, 64), 4),
              ((992, 2080, 2176), (96, 128), 4), ((1504, 2080, 4096), (128, 128), 4)]


@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("shape,tile,split", FEW_TOKENS, ids=["x".join(map(str, c[0])) for c in FEW_TOKENS])
def test_weight_slabs_with_few_tokens(shape, tile, split, fmt_name):
    (M, N, K), seed = shape, 5
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    if fmt_name == "nvfp4" or M <= 320:
        assert nv.gemm_tile(M, N, K, fmt) == tile and nv.gemm_split(M, N, K, fmt) == split
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W, dY = (torch.randn(s, generator=g, device="cuda") for s in ((M, K), (N, K), (M, N)))
    print(f"[case] weight slabs {fmt_name} {M}x{N}x{K}", flush=True)
    wq = nv.quantize_weight(W, M, fmt)
    saved = torch.empty(nv.linear_saved_bytes(M, N, K, fmt), dtype=torch.uint8, device="cuda")
    for out_dtype in (torch.float32, torch.bfloat16):
        Y = nv.linear_fwd(X, None, fmt, out_dtype, w_operands=wq, N=N, saved=saved, bwd_seed=seed)
        assert torch.equal(Y, nv.linear_fwd(X, W, fmt, out_dtype))
    got = nv.linear_bwd(dY, None, None, seed, fmt, saved=saved, K=K, w_operands=wq)
    for a, b in zip(got, nv.linear_bwd(dY, X, W, seed, fmt)):
        assert torch.equal(a, b)


# bf16 X and W of together more than 512 quantizer tiles (128 x 256) are one run of tiles over both tensors: the change from X to W in a
# workgroup's first, second and third tile, tiles past the edges of both; row-major and slabs; the bits of the calls that quantize alone.
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("M,N,K", [(160, 8224, 4224), (2080, 4128, 4224), (12320, 288, 2176), (23328, 416, 2336)])
def test_saved_operands_of_many_tiles(M, N, K, fmt_name):
    seed = 11
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W, dY = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((M, K), (N, K), (M, N)))
    W *= 0.02
    print(f"[case] saved operands of many tiles {fmt_name} {M}x{N}x{K}", flush=True)
    saved = torch.empty(nv.linear_saved_bytes(M, N, K, fmt), dtype=torch.uint8, device="cuda")
    Y = nv.linear_fwd(X, W, fmt, saved=saved, bwd_seed=seed)
    assert torch.equal(Y, nv.linear_fwd(X, W, fmt))
    got = nv.linear_bwd(dY, None, None, seed, fmt, saved=saved, K=K)
    for a, b in zip(got, nv.linear_bwd(dY, X, W, seed, fmt)):
        assert torch.equal(a, b)


# A backward call that has neither W^T nor X^T quantizes all three tensors in one launch where they are small: on the lines of that
# (4M elements of dY, 8M of bf16 W and X, 16M of binary32) and past them, one of the three past, odd sizes; maxima taken, scales handed
# over, W's operands at hand.  The bits of the separate calls.
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4", "e4m3_32", "e4m3_64"])
@pytest.mark.parametrize("shape", [(64, 64, 64), (192, 320, 1088), (1056, 416, 2080), (2048, 2048, 64), (2048, 2112, 64), (64, 2048, 4096), (64, 2112, 4096),
                                   (2112, 64, 4096)])
def test_small_tensors_of_a_backward_call(shape, fmt_name, dtype):
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    M, N, K = (-(-n // max(block, 32)) * max(block, 32) for n in shape)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    X, W, dY = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((M, K), (N, K), (M, N)))
    seed = 21
    print(f"[case] small backward {fmt_name} {M}x{N}x{K} {dtype}", flush=True)
    dX = nv.gemm(nv.quantize(dY, 1, nv.SR, seed, fmt), nv.quantize(W, 0, nv.RTN, 0, fmt), fmt)
    dW = nv.gemm(nv.quantize(dY, 0, nv.SR, seed + 1, fmt), nv.quantize(X, 0, nv.SR, seed + 2, fmt), fmt)
    scales = torch.empty(2, device="cuda")
    nv.linear_fwd(X, W, fmt, scales_out=scales)
    for kw in ({}, dict(xw_scales=scales), dict(w_operands=nv.quantize_weight(W, M, fmt))):
        got = nv.linear_bwd(dY, X, W, seed, fmt, **kw)
        assert torch.equal(got[0], dX) and torch.equal(got[1], dW), list(kw)


# MXFP4 tensors of up to 4M elements keep their rows in training calls whose products could take slabs (contractions of 512 and more): on
# that line and past it, one operand on each side of it, operands handed over by the forward call.
@pytest.mark.parametrize("shape", [(512, 512, 512), (96, 1024, 640), (2048, 2048, 2048), (2048, 2080, 2048), (2080, 512, 2048), (512, 2080, 2048)])
def test_small_mxfp4_training_tensors(shape):
    M, N, K = shape
    fmt, seed = nv.MXFP4, 9
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    X, W, dY = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((M, K), (N, K), (M, N)))
    print(f"[case] small MXFP4 training {M}x{N}x{K}", flush=True)
    Yr = nv.gemm(nv.quantize(X, fmt=fmt), nv.quantize(W, fmt=fmt), fmt)
    dX = nv.gemm(nv.quantize(dY, 1, nv.SR, seed, fmt), nv.quantize(W, 0, nv.RTN, 0, fmt), fmt)
    dW = nv.gemm(nv.quantize(dY, 0, nv.SR, seed + 1, fmt), nv.quantize(X, 0, nv.SR, seed + 2, fmt), fmt)
    wq = nv.quantize_weight(W, M, fmt)
    for kw in ({}, dict(w_operands=wq)):
        saved = torch.empty(nv.linear_saved_bytes(M, N, K, fmt), dtype=torch.uint8, device="cuda")
        Y = nv.linear_fwd(X, None if kw else W, fmt, saved=saved, bwd_seed=seed, N=N, **kw)
        got = nv.linear_bwd(dY, None, None, seed, fmt, saved=saved, K=K, **kw)
        for a, b in zip((Y, *got), (Yr, dX, dW)):
            assert torch.equal(a, b), list(kw)


# 160 x 256, whose upper four waves have 96 rows and whose lower four 64: whole tiles, one row or column past a tile and past the upper
# waves' rows, rows that reach into the next slab, whole contractions and K tails.
UNEVEN = [(777, 12288, 1024), (961, 8193, 1056), (1537, 6144, 1088), (2399, 3841, 1184), (320, 32768, 1024), (1600, 6144, 1152)]


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "e4m3_32", "e4m3_128"])
@pytest.mark.parametrize("shape", UNEVEN, ids=["x".join(map(str, s)) for s in UNEVEN])
def test_uneven_waves_sampled(shape, fmt_name, out_dtype):
    block, scale = FORMATS[fmt_name]
    M, N, K = shape
    K = -(-K // block) * block
    assert nv.gemm_tile(M, N, K, nv.Format(block, scale, 1)) == (160, 256)
    check_sampled((M, N, K), fmt_name, out_dtype)


@pytest.mark.parametrize("shape", [(784, 12288, 1024), (2384, 3840, 1152)])
def test_uneven_waves_across_slabs(shape):
    M, N, K = shape
    assert nv.gemm_tile(M, N, K) == (160, 256)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W = (torch.randn((n, K), generator=g, device="cuda") for n in (M, N))
    print(f"[case] gemm uneven tiles across slabs {M}x{N}x{K}", flush=True)
    ops = [(nv.quantize_dual(t)[0], nv.quantize_dual(t, slab_rows=True)[0]) for t in (X, W)]
    plain = nv.gemm(ops[0][0], ops[1][0], shape=shape)
    for slabs in ((True, False), (False, True), (True, True)):
        assert torch.equal(nv.gemm(ops[0][slabs[0]], ops[1][slabs[1]], slabs=slabs, shape=shape), plain), slabs


# 128 x 256 with two groups of waves: an even and an odd number of K tiles (the second group's last one is zeros), K tails, edges.
TWO_GROUPS = [(2048, 4096, 2048), (2000, 4001, 2944), (1921, 3841, 2912), (1793, 4096, 2272), (900, 8192, 3168)]


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "e4m3_32", "e4m3_64"])
@pytest.mark.parametrize("shape", TWO_GROUPS, ids=["x".join(map(str, s)) for s in TWO_GROUPS])
def test_two_groups_sampled(shape, fmt_name, out_dtype):
    block, scale = FORMATS[fmt_name]
    M, N, K = shape
    K = -(-K // block) * block
    assert nv.gemm_tile(M, N, K) == (128, 256) and nv.gemm_split(M, N, K) == 2
    check_sampled((M, N, K), fmt_name, out_dtype)


@pytest.mark.parametrize("shape", [(2048, 4096, 2944), (2032, 4080, 2048)])
def test_two_groups_on_slabs(shape):
    M, N, K = shape
    assert nv.gemm_split(M, N, K) == 2
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W = (torch.randn((n, K), generator=g, device="cuda") for n in (M, N))
    print(f"[case] gemm two groups on slabs {M}x{N}x{K}", flush=True)
    ops = [(nv.quantize_dual(t)[0], nv.quantize_dual(t, slab_rows=True)[0]) for t in (X, W)]
    plain = nv.gemm(ops[0][0], ops[1][0], shape=shape)
    for slabs in ((True, False), (False, True), (True, True)):
        assert torch.equal(nv.gemm(ops[0][slabs[0]], ops[1][slabs[1]], slabs=slabs, shape=shape), plain), slabs
