"""Linear layers of a small network, whose forward and backward calls are one launch each (fused_small.hip): the bits of the separate
quantizers and products.  One tile and many, K tails, the longest contractions and the largest tensors that are fused and the next longer
ones, calls in which only one direction is."""
import pytest
import torch

pytestmark = pytest.mark.gpu

nv = None


@pytest.fixture(scope="module", autouse=True)
def _binding():
    global nv
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2505_19115_amd import binding
    nv = binding
    yield


FORMATS = {"nvfp4": (16, 0, 1), "mxfp4": (32, 1, 0), "nvfp4_unscaled": (16, 0, 0)}
# binary32 tensors of 128 KB: 64 x 512, 256 x 128; the backward call takes 256 tokens, contractions reach 512
SHAPES = [(32, 32, 32), (64, 256, 128), (96, 160, 64), (160, 96, 224), (64, 512, 64), (64, 544, 64), (64, 64, 512), (32, 64, 544), (256, 128, 128), (256, 64, 96),
          (288, 64, 96), (512, 64, 64), (544, 32, 32), (128, 256, 128), (128, 288, 128), (224, 32, 128), (32, 480, 32), (64, 512, 128), (256, 256, 256)]


def tensors(M, N, K, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    X, W, dY = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((M, K), (N, K), (M, N)))
    X.view(-1)[-1], W.view(-1)[0], dY.view(-1)[M * N // 2] = 9.0, -7.0, 11.0  # (the tensors' maxima, one per place)
    return X, W, dY


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt_name", FORMATS)
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_layer_in_one_launch_per_call(shape, fmt_name, dtype):
    (M, N, K), fmt, seed = shape, nv.Format(*FORMATS[fmt_name]), 13
    X, W, dY = tensors(M, N, K, dtype, M + N + K)
    print(f"[case] fused layer {fmt_name} {M}x{N}x{K} {dtype}", flush=True)
    Xq, Wq = nv.quantize(X, fmt=fmt), nv.quantize(W, fmt=fmt)
    for out_dtype in (torch.float32, torch.bfloat16):
        Y = nv.gemm(Xq, Wq, fmt, out_dtype)
        dX = nv.gemm(nv.quantize(dY, 1, nv.SR, seed, fmt), nv.quantize(W, 0, nv.RTN, 0, fmt), fmt, out_dtype)
        dW = nv.gemm(nv.quantize(dY, 0, nv.SR, seed + 1, fmt), nv.quantize(X, 0, nv.SR, seed + 2, fmt), fmt, out_dtype)
        saved = torch.full((nv.linear_saved_bytes(M, N, K, fmt),), 0xA5, dtype=torch.uint8, device="cuda")
        scales = torch.zeros(2, device="cuda")
        assert torch.equal(nv.linear_fwd(X, W, fmt, out_dtype, saved=saved, bwd_seed=seed, scales_out=scales), Y)
        assert float(scales[0]) == float(Xq[2]) and float(scales[1]) == float(Wq[2])
        assert torch.equal(nv.linear_fwd(X, W, fmt, out_dtype), Y)
        got = nv.linear_bwd(dY, None, None, seed, fmt, out_dtype, saved=saved, K=K)
        assert torch.equal(got[0], dX) and torch.equal(got[1], dW)
        # the weights' operands written beforehand, and one gradient alone
        wq, saved_x = nv.quantize_weight(W, M, fmt), torch.empty_like(saved)
        assert torch.equal(nv.linear_fwd(X, None, fmt, out_dtype, saved=saved_x, bwd_seed=seed, w_operands=wq, N=N), Y)
        got = nv.linear_bwd(dY, None, None, seed, fmt, out_dtype, saved=saved_x, K=K, w_operands=wq)
        assert torch.equal(got[0], dX) and torch.equal(got[1], dW)


# Both sides of the lines that the numbers of workgroups draw (test_host_logic.py): one round of them, the second round of few rows, separate calls.
@pytest.mark.parametrize("shape,dtype,fmt_name", [((480, 512, 64), torch.bfloat16, "nvfp4"), ((512, 512, 64), torch.bfloat16, "nvfp4"), ((512, 544, 64), torch.bfloat16, "nvfp4"),
                                                  ((1024, 512, 32), torch.float32, "nvfp4"), ((128, 128, 288), torch.bfloat16, "nvfp4"), ((1024, 800, 64), torch.bfloat16, "mxfp4"),
                                                  ((1024, 992, 64), torch.bfloat16, "mxfp4"), ((128, 128, 1344), torch.bfloat16, "nvfp4"), ((128, 128, 1376), torch.bfloat16, "nvfp4"),
                                                  ((256, 256, 704), torch.bfloat16, "mxfp4"), ((64, 512, 832), torch.float32, "nvfp4"), ((128, 128, 2720), torch.bfloat16, "mxfp4")])
def test_layers_beside_the_lines(shape, dtype, fmt_name):
    test_layer_in_one_launch_per_call(shape, fmt_name, dtype)


@pytest.mark.parametrize("fmt_name", FORMATS)
@pytest.mark.parametrize("M,N,K", [(17, 70, 96), (33, 33, 160), (63, 100, 512), (127, 31, 32), (200, 1, 64)])
def test_ragged_forward(M, N, K, fmt_name):
    fmt = nv.Format(*FORMATS[fmt_name])
    X, W, _ = tensors(M, N, K, torch.float32, M)
    print(f"[case] fused forward {fmt_name} {M}x{N}x{K}", flush=True)
    assert torch.equal(nv.linear_fwd(X, W, fmt), nv.gemm(nv.quantize(X, fmt=fmt), nv.quantize(W, fmt=fmt), fmt))


def test_buffer_of_another_call_poisons_the_gradients():
    M, N, K, seed = 64, 256, 128, 3
    X, W, dY = tensors(M, N, K, torch.float32, 1)
    saved = torch.empty(nv.linear_saved_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    nv.linear_fwd(X, W, saved=saved, bwd_seed=seed)
    with pytest.raises(nv.Nvfp4Error):
        nv.linear_bwd(dY, None, None, seed + 1, saved=saved, K=K)
    moved = torch.empty(saved.numel() + 1280, dtype=torch.uint8, device="cuda")[1280:].copy_(saved)  # an address that no forward call wrote to
    good, bad = nv.linear_bwd(dY, None, None, seed, saved=moved, K=K), nv.linear_bwd(dY, None, None, seed + 1, saved=moved, K=K)
    assert all(torch.isfinite(t).all() for t in good) and all(torch.isnan(t).all() for t in bad)


def test_layer_in_a_graph():
    M, N, K, seed = 64, 256, 128, 5
    X, W, dY = tensors(M, N, K, torch.float32, 2)
    ws = [torch.empty(f(M, N, K, nv.C.byref(nv.NVFP4.c())), dtype=torch.uint8, device="cuda")
          for f in (nv.lib.nvfp4_linear_fwd_workspace_bytes, nv.lib.nvfp4_linear_bwd_workspace_bytes)]
    saved = torch.empty(nv.linear_saved_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    Y, dX, dW = (torch.empty(s, device="cuda") for s in ((M, N), (M, K), (N, K)))

    def layer(out, grads, buffer):
        nv.linear_fwd(X, W, workspace=ws[0], out=out, saved=buffer, bwd_seed=seed)
        nv.linear_bwd(dY, None, None, seed, workspace=ws[1], out=grads, saved=buffer, K=K)

    layer(Y, (dX, dW), saved)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer(Y, (dX, dW), saved)
    eager = [torch.empty_like(t) for t in (Y, dX, dW)]
    for i in range(4):
        for t, s in zip((X, W, dY), tensors(M, N, K, torch.float32, 20 + i)):
            t.copy_(s)
        graph.replay()
        layer(eager[0], (eager[1], eager[2]), torch.empty_like(saved))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((Y, dX, dW), eager)), i
