"""Calls that bring no workspace take a block of the caching allocator for their launches and give it back behind them: the same bits as with a workspace
of the caller's, on another stream, and captured into a graph that is replayed between eager calls; nothing stays allocated."""
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


def tensors(M, N, K):
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    return [torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((M, K), (N, K), (M, N))]


def calls(X, W, dY, fmt, work=None):
    f = nv.linear_fwd(X, W, fmt, workspace=work)
    q = nv.quantize(dY, 1, nv.SR, 5, fmt)
    return [f, *nv.linear_bwd(dY, X, W, 7, fmt, workspace=work), *q, nv.quant_noise(dY, q, 1, fmt)]


@pytest.mark.parametrize("fmt_name", ["NVFP4", "MXFP4"])
@pytest.mark.parametrize("shape", [(64, 96, 128), (512, 1024, 768)])
def test_blocks_for_a_call(shape, fmt_name):
    fmt = getattr(nv, fmt_name)
    X, W, dY = tensors(*shape)
    print(f"[case] blocks for a call {shape} {fmt_name}", flush=True)
    want = calls(X, W, dY, fmt, torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            got = calls(X, W, dY, fmt)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        del got
        assert torch.cuda.memory_allocated() == before


def test_blocks_in_a_graph():
    X, W, dY = tensors(256, 512, 384)
    print("[case] blocks in a graph", flush=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls(X, W, dY, nv.NVFP4)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        Y = nv.linear_fwd(X, W, nv.NVFP4)
        dX, dW = nv.linear_bwd(dY, X, W, 7, nv.NVFP4)
    for i in range(4):
        X.mul_(-0.5 if i % 2 else 1.5)
        graph.replay()
        torch.cuda.synchronize()
        want = calls(X, W, dY, nv.NVFP4)
        torch.cuda.synchronize()
        assert torch.equal(Y, want[0]) and torch.equal(dX, want[1]) and torch.equal(dW, want[2]), i


@pytest.mark.parametrize("lacking", ["_raw_alloc", "_raw_delete", "_raw_device"])
def test_tensors_where_torch_has_no_raw_entry(lacking, monkeypatch):
    X, W, dY = tensors(64, 96, 128)
    print(f"[case] tensors for a call, without {lacking}", flush=True)
    want = calls(X, W, dY, nv.NVFP4, torch.empty(1 << 20, dtype=torch.uint8, device="cuda"))
    monkeypatch.setattr(nv, lacking, None)
    got = calls(X, W, dY, nv.NVFP4)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
