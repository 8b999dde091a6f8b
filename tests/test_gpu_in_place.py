"""Outputs of linear calls on the memory of an input, at sizes whose calls are one launch otherwise: whole tensors, parts of them, and the
two sides next to each other.  The bits of the same call with an output of its own."""
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


def normal(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda")


def on_memory_of(t, elements, shape, dtype, offset):
    """(a copy of t and an output of `shape` that starts `offset` bytes behind the copy's first byte, in one buffer)"""
    size, out = t.numel() * t.element_size(), elements * dtype.itemsize
    buffer = torch.zeros(max(size, offset + out), dtype=torch.uint8, device="cuda")
    copy = buffer[:size].view(t.dtype).view(t.shape).copy_(t)
    return copy, buffer[offset:offset + out].view(dtype).view(shape)


@pytest.mark.parametrize("fmt_name", ["NVFP4", "MXFP4"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,N,K", [(1, 4096, 4096), (2, 2048, 2048), (16, 320, 320), (64, 128, 128), (64, 256, 128)])
def test_output_on_the_activation(M, N, K, dtype, fmt_name):
    fmt = getattr(nv, fmt_name)
    X, W = normal(M, M, K).to(dtype), normal(N, N, K).to(dtype)
    for wq in (None, nv.quantize_weight(W, M, fmt)):
        weight = dict(W=W) if wq is None else dict(W=None, w_operands=wq, N=N)
        for out_dtype in (torch.bfloat16, torch.float32):
            want = nv.linear_fwd(X, fmt=fmt, out_dtype=out_dtype, **weight)
            size = X.numel() * X.element_size()
            for offset in (0, 256, size - 16, size):
                print(f"[case] Y on X {fmt_name} {M}x{N}x{K} {dtype} {out_dtype} packed={wq is not None} offset={offset}", flush=True)
                x, y = on_memory_of(X, M * N, (M, N), out_dtype, offset)
                nv.linear_fwd(x, fmt=fmt, out=y, **weight)
                assert torch.equal(y, want), (offset, out_dtype)


@pytest.mark.parametrize("fmt_name", ["NVFP4", "MXFP4"])
def test_output_on_the_weight_and_gradients_on_the_upstream_one(fmt_name):
    fmt, seed = getattr(nv, fmt_name), 3
    M = N = K = 128
    X, W, dY = normal(1, M, K), normal(2, N, K), normal(3, M, N)
    want = nv.linear_fwd(X, W, fmt)
    w, y = on_memory_of(W, M * N, (M, N), torch.float32, 0)
    print(f"[case] Y on W, dX and dW on dY {fmt_name}", flush=True)
    nv.linear_fwd(X, w, fmt, out=y)
    assert torch.equal(y, want)
    saved = torch.empty(nv.linear_saved_bytes(M, N, K, fmt), dtype=torch.uint8, device="cuda")
    w, y = on_memory_of(W, M * N, (M, N), torch.float32, 0)
    nv.linear_fwd(X, w, fmt, out=y, saved=saved, bwd_seed=seed)
    assert torch.equal(y, want)
    dX, dW = nv.linear_bwd(dY, None, None, seed, fmt, saved=saved, K=K)
    for which in (0, 1):
        dy, grad = on_memory_of(dY, M * K, (M, K), torch.float32, 0)
        own = torch.empty_like(dX)
        nv.linear_bwd(dy, None, None, seed, fmt, saved=saved, K=K, out=(grad, own) if which == 0 else (own, grad))
        assert torch.equal(grad, (dX, dW)[which]) and torch.equal(own, (dX, dW)[1 - which])
