"""Products of up to 16 rows (gemm_thin.hip): one K tile, less, remainders of the waves' K tiles and of the stages in flight, K tails, rows
and columns past the edge, each number of columns per workgroup and of waves, row-major operands and slabs, outputs of odd pitch; and calls
that quantize a small activation in the same launch, at the edges of what it takes.  Against the fp64 oracle and the separate calls."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import ofmt, to_np
from test_gpu_gemm_tiles import FORMATS, close, operand

pytestmark = pytest.mark.gpu

nv = None


@pytest.fixture(scope="module", autouse=True)
def _binding():
    global nv
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2505_19115_amd import binding
    nv = binding
    yield


# columns per workgroup 16 (N to 4096), 32 (to 8192), 48 (to 12288), 64; 8 waves, and 16 from K = 2048 (NVFP4) and 8192 (MXFP4) on
SHAPES = [(1, 1, 32), (16, 16, 128), (15, 17, 96), (16, 4096, 160), (3, 40, 1024), (7, 75, 1152), (16, 100, 2048), (9, 33, 2080), (2, 48, 8192),
          (16, 50, 8224), (16, 4097, 288), (5, 8192, 2176), (12, 8193, 1056), (16, 12280, 2112), (1, 12289, 544), (16, 16384, 2240), (4, 16385, 512)]


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_few_rows(shape, fmt_name, out_dtype):
    block, scale = FORMATS[fmt_name]
    M, N, K = shape
    fmt = nv.Format(block, scale, 1 - scale)
    rng = np.random.default_rng(M + 7 * N + K)
    A, B = operand(rng, M, K, block, scale), operand(rng, N, K, block, scale)
    dev = lambda o: (torch.from_numpy(o[0]).cuda(), torch.from_numpy(o[1]).cuda(), torch.tensor([o[2]], dtype=torch.float32, device="cuda"))
    of = ofmt(fmt)
    ref, ref_abs = oracle.gemm_nt(A, B, of), oracle.gemm_nt(A, B, of, take_abs=True)
    for ld in (N, -(-N // 4) * 4 + 4, (N | 1) + 2):
        print(f"[case] thin {fmt_name} {M}x{N}x{K} ldc={ld} {out_dtype}", flush=True)
        out = torch.full((M, ld), -1.0, device="cuda", dtype=out_dtype)
        nv.gemm(dev(A), dev(B), fmt, out=out[:, :N])
        torch.cuda.synchronize()
        close(to_np(out[:, :N].float()), ref, ref_abs, f"ldc {ld}", out_dtype)
        assert bool((out[:, N:] == -1.0).all()), "columns outside the output were written"


@pytest.mark.parametrize("fmt_name,shape", [("nvfp4", (16, 32800, 1152)), ("nvfp4", (13, 32768, 2176)), ("mxfp4", (16, 300, 512)), ("mxfp4", (3, 8448, 640)),
                                            ("mxfp4", (16, 2080, 8320))])
def test_few_rows_in_slabs(fmt_name, shape):
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W = (torch.randn((-(-n // block) * block, K), generator=g, device="cuda") for n in (M, N))
    ops = [(nv.quantize_dual(t, fmt=fmt)[0], nv.quantize_dual(t, fmt=fmt, slab_rows=True)[0]) for t in (X, W)]
    print(f"[case] thin slabs {fmt_name} {M}x{N}x{K}", flush=True)
    plain = nv.gemm(ops[0][0], ops[1][0], fmt, shape=shape)
    for slabs in ((True, False), (False, True), (True, True)):
        assert torch.equal(nv.gemm(ops[0][slabs[0]], ops[1][slabs[1]], fmt, slabs=slabs, shape=shape), plain), slabs


# The activation quantized by the kernel: up to 24 KB of it (on the line, one row past it), weights row-major and in slabs; the codes are
# those of the quantizer, so the bits are those of the separate calls.  Tensors with a largest element at either end, zeros, one huge element.
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", ["nvfp4", "mxfp4"])
@pytest.mark.parametrize("shape", [(1, 32, 32), (16, 4128, 32), (16, 2080, 768), (16, 96, 384), (3, 4128, 4096), (3, 1056, 2048), (1, 8224, 2080), (1, 2080, 12288),
                                   (1, 512, 6144), (2, 12320, 4128), (7, 416, 416), (1, 16416, 640), (4, 1024, 4096)])
def test_activation_quantized_with_the_product(shape, fmt_name, dtype):
    block, scale = FORMATS[fmt_name]
    fmt = nv.Format(block, scale, 1 - scale)
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(dtype)
    wq, Wq = nv.quantize_weight(W, M, fmt), nv.quantize(W, fmt=fmt)
    for kind in ("normal", "first", "last", "zero", "huge"):
        X = torch.randn((M, K), generator=g, device="cuda")
        if kind in ("first", "last"):
            X.view(-1)[0 if kind == "first" else -1] = -40.0
        X = (X * {"zero": 0.0, "huge": 1e30}.get(kind, 1.0)).to(dtype)
        print(f"[case] thin with quantizer {fmt_name} {M}x{N}x{K} {dtype} {kind}", flush=True)
        scales = torch.zeros(2, device="cuda")
        for out_dtype in (torch.float32, torch.bfloat16):
            Y = nv.linear_fwd(X, None, fmt, out_dtype, w_operands=wq, N=N, scales_out=scales)
            Xq = nv.quantize(X, fmt=fmt)
            assert torch.equal(Y, nv.gemm(Xq, Wq, fmt, out_dtype)), (kind, out_dtype)
            assert float(scales[0]) == float(Xq[2]) and float(scales[1]) == float(Wq[2])
        assert torch.equal(nv.linear_fwd(X, W, fmt, torch.bfloat16), Y)


def test_decode_call_in_a_graph():
    M, N, K = 2, 4096, 4096
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    W = torch.randn((N, K), generator=g, device="cuda").bfloat16()
    X, Y = torch.zeros((M, K), device="cuda", dtype=torch.bfloat16), torch.zeros((M, N), device="cuda", dtype=torch.bfloat16)
    wq = nv.quantize_weight(W, M)
    ws = torch.empty(nv.lib.nvfp4_linear_fwd_workspace_bytes(M, N, K, nv.C.byref(nv.NVFP4.c())), dtype=torch.uint8, device="cuda")
    call = lambda: nv.linear_fwd(X, None, out_dtype=torch.bfloat16, w_operands=wq, N=N, workspace=ws, out=Y)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in range(4):
        X.copy_(torch.randn((M, K), generator=g, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, nv.gemm(nv.quantize(X), nv.quantize(W), out_dtype=torch.bfloat16)), i
