"""Columns and both orientations of small tensors in blocks of 64 and 128, whose kernels give a block to two or four waves: bit for bit what
the general kernels write (selected by the software formulation of the rounding) and, for sizes that are cheap there, the oracle.  One
block, numbers of blocks that do not fill a workgroup, columns that do not fill a wave, row pitches, the largest such tensor and the
next one, tensors with and without a scale, zeros, one huge element."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import ofmt

pytestmark = pytest.mark.gpu

nv = None


@pytest.fixture(scope="module", autouse=True)
def _binding():
    global nv
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2505_19115_amd import binding
    nv = binding
    yield


def general(call):
    before = nv.cross_check_switches()
    nv.cross_check_switches(nv.SWITCH_SOFT_CONVERT)
    try:
        return call()
    finally:
        nv.cross_check_switches(before)


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


SHAPES = [(1, 8), (1, 72), (3, 128), (5, 200), (9, 64), (2, 1000), (16, 136)]  # blocks down the columns, columns


@pytest.mark.parametrize("scaled", [0, 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("blocks,cols", SHAPES)
def test_columns(blocks, cols, block, dtype, scaled):
    rows, fmt = blocks * block, nv.Format(block, 0, scaled)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + cols)
    print(f"[case] wide columns {rows}x{cols} block {block} {dtype} scaled {scaled}", flush=True)
    for pad in (0, 8, 64):
        x = torch.randn((rows, cols + pad), generator=g, device="cuda")
        x[rows // 2, cols // 2] = 1e4
        x[:block, 0] = 0.0
        x = x.to(dtype)[:, :cols]
        for rounding in (nv.RTN, nv.SR):
            got = nv.quantize(x, 0, rounding, 77, fmt)
            assert same(got, general(lambda: nv.quantize(x, 0, rounding, 77, fmt))), (pad, rounding)
            if rows * cols <= 1 << 17:
                ref = oracle.quantize(x.contiguous().cpu(), 0, rounding, 77, ofmt(fmt))
                assert np.array_equal(got[0].cpu().numpy(), ref[0]) and np.array_equal(got[1].cpu().numpy(), ref[1]) and float(got[2].item()) == ref[2]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("rows,cols", [(128, 128), (384, 640), (1152, 384), (2048, 4096), (2048, 4224), (8192, 1024)])
def test_both_orientations(rows, cols, block, dtype):
    fmt = nv.Format(block, 0, 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    x = (torch.randn((rows, cols), generator=g, device="cuda") * 1e-3).to(dtype)
    print(f"[case] wide dual {rows}x{cols} block {block} {dtype}", flush=True)
    for rnd_r, rnd_c in ((nv.RTN, nv.RTN), (nv.RTN, nv.SR), (nv.SR, nv.SR), (nv.SR, nv.RTN)):
        got = nv.quantize_dual(x, rnd_r, 5, rnd_c, 6, fmt)
        ref = general(lambda: nv.quantize_dual(x, rnd_r, 5, rnd_c, 6, fmt))
        assert same(got[0], ref[0]) and same(got[1], ref[1]), (rnd_r, rnd_c)


# layers whose tensors are small in all three places, in some, in none; every hand-over
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("shape", [(128, 128, 128), (384, 256, 640), (4096, 2176, 256), (2048, 4224, 128), (256, 2176, 4096), (2176, 256, 4096)])
def test_layers(shape, block, dtype):
    (M, N, K), fmt, seed = shape, nv.Format(block, 0, 1), 31
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(shape))
    X, W, dY = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((M, K), (N, K), (M, N)))
    print(f"[case] wide layer {shape} block {block} {dtype}", flush=True)
    Y = nv.gemm(nv.quantize(X, fmt=fmt), nv.quantize(W, fmt=fmt), fmt)
    dX = nv.gemm(nv.quantize(dY, 1, nv.SR, seed, fmt), nv.quantize(W, 0, nv.RTN, 0, fmt), fmt)
    dW = nv.gemm(nv.quantize(dY, 0, nv.SR, seed + 1, fmt), nv.quantize(X, 0, nv.SR, seed + 2, fmt), fmt)
    wq, scales = nv.quantize_weight(W, M, fmt), torch.empty(2, device="cuda")
    saved = torch.empty(nv.linear_saved_bytes(M, N, K, fmt), dtype=torch.uint8, device="cuda")
    for kw in ({}, dict(w_operands=wq)):
        assert torch.equal(nv.linear_fwd(X, None if kw else W, fmt, saved=saved, bwd_seed=seed, N=N, scales_out=scales, **kw), Y)
        got = nv.linear_bwd(dY, None, None, seed, fmt, saved=saved, K=K, **kw)
        assert torch.equal(got[0], dX) and torch.equal(got[1], dW), ("saved", list(kw))
        # written for another seed: NaN from an address that the host has no record of (one that an earlier test's call wrote to is refused)
        moved = torch.empty(saved.numel() + 768, dtype=torch.uint8, device="cuda")[768:].copy_(saved)
        try:
            assert all(torch.isnan(t).all() for t in nv.linear_bwd(dY, None, None, seed + 1, fmt, saved=moved, K=K, **kw))
        except nv.Nvfp4Error as e:
            assert e.code == nv.EINVAL
        got = nv.linear_bwd(dY, X, W, seed, fmt, xw_scales=scales, **kw)
        assert torch.equal(got[0], dX) and torch.equal(got[1], dW), ("scales", list(kw))
