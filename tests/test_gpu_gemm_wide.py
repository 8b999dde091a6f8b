"""E4M3 products on four waves of 128 columns (contractions of more than seven K tiles): every tile with whole contractions and K tails, an even and an odd
number of K tiles, rows and columns past the edge; and outputs that two kinds of tiles share (whole rounds of 256 x 256, smaller ones for the rest)."""
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


BLOCKS = (16, 32, 64, 128)

# (shape, tile, groups): K in blocks of 32 is rounded up to the block size, which turns a tail of 32 into one of 64 or a whole K tile
TILES = [((5975, 1281, 928), (160, 256), 1), ((8280, 903, 1024), (160, 256), 1), ((901, 8699, 928), (192, 256), 1), ((1320, 5904, 1152), (192, 256), 1),
         ((3720, 3219, 928), (256, 256), 1), ((1820, 6530, 1024), (256, 256), 1), ((8204, 580, 1472), (128, 256), 2), ((841, 5838, 1536), (128, 256), 2)]

# whole rounds of 256 x 256, then 192 x 256 for the last tile columns, for the last tile rows, 128 x 256 in two groups for the same
MIXED = [((1796, 13201, 2304), "columns, 192"), ((2313, 10244, 2432), "rows, 192"), ((2696, 13396, 2304), "columns, two groups"), ((11795, 3084, 2432), "rows, two groups")]


def assert_mixed(M, N, K, which):
    """The library takes this division (and the tests of two kinds of tiles reach the kernel that they name)."""
    mix = nv.gemm_mixed(M, N, K)
    assert mix is not None and mix["rows"] == which.startswith("rows") and (mix["tile"], mix["groups"]) == (((192, 256), 1) if "192" in which else ((128, 256), 2)), (mix, which)


def operand(rng, rows, K, block):
    return (rng.integers(0, 256, (rows, K // 2)).astype(np.uint8), rng.integers(0x01, 0x7F, (rows, K // block)).astype(np.uint8), 0.75)


def check(shape, block, out_dtype):
    M, N, K = shape
    fmt = nv.Format(block, nv.SCALE_E4M3, 1)
    rng = np.random.default_rng(M + 7 * N + K)
    A, B = operand(rng, M, K, block), operand(rng, N, K, block)
    print(f"[case] wide products {M}x{N}x{K} blocks of {block} {out_dtype}", flush=True)
    dev = [(torch.from_numpy(o[0]).cuda(), torch.from_numpy(o[1]).cuda(), torch.tensor([o[2]], dtype=torch.float32, device="cuda")) for o in (A, B)]
    out = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    nv.gemm(*dev, fmt, out=out)
    torch.cuda.synchronize()
    assert not bool(out.isnan().any()), "outputs that nobody wrote"
    got = to_np(out.float())
    # random outputs, and those around every multiple of 32 rows and columns at both ends
    edge = lambda n: np.unique(np.clip(np.concatenate([np.arange(0, 520, 32) - 1, np.arange(0, 520, 32), n - 1 - np.arange(0, 520, 32), [n - 2]]), 0, n - 1))
    ii = np.concatenate([rng.integers(0, M, 3000), np.repeat(edge(M), 40), rng.integers(0, M, 40 * len(edge(N)))])
    jj = np.concatenate([rng.integers(0, N, 3000), rng.integers(0, N, 40 * len(edge(M))), np.repeat(edge(N), 40)])
    of = ofmt(fmt)
    (assert_bf16_gemm_close if out_dtype == torch.bfloat16 else assert_gemm_close)(
        got[ii, jj], oracle.gemm_nt_sample(A, B, ii, jj, of), oracle.gemm_nt_sample(A, B, ii, jj, of, take_abs=True), f"{shape} {block}")
    return dev, fmt, out


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("shape,tile,groups", TILES, ids=["x".join(map(str, s)) for s, _, _ in TILES])
def test_tiles(shape, tile, groups, block, out_dtype):
    M, N, K = shape
    assert nv.gemm_tile(M, N, K) == tile and nv.gemm_split(M, N, K) == groups
    check((M, N, -(-K // block) * block), block, out_dtype)


@pytest.mark.parametrize("block,out_dtype", [(16, torch.bfloat16), (16, torch.float32), (32, torch.float32), (64, torch.bfloat16), (128, torch.float32)])
@pytest.mark.parametrize("shape,which", MIXED, ids=[f"{'x'.join(map(str, s))}: {n}" for s, n in MIXED])
def test_two_kinds_of_tiles(shape, which, block, out_dtype):
    M, N, K = shape
    assert_mixed(M, N, K, which)
    assert nv.gemm_tile(M, N, K) == (256, 256) and -(-M // 256) * -(-N // 256) % 256 and -(-M // 256) * -(-N // 256) > 256
    (A, B, fmt, whole) = (lambda d, f, o: (*d, f, o))(*check(shape, block, out_dtype))
    if out_dtype == torch.float32:
        # every output against the same rows by themselves (592 at a time: scale rows stay aligned), which other tiles compute.  Both are binary32 sums of K exact products: each is at most
        # K 2^-24 sum |a b| from the true one, and that sum at most the product of the two rows' norms.
        norm = lambda o: nv.gemm(o, o, fmt).diagonal().sqrt() if o[0].shape[0] <= 592 else torch.cat([norm((o[0][i:i + 592], o[1][i:i + 592], o[2])) for i in range(0, o[0].shape[0], 592)])
        nA, nB = norm(A), norm(B)
        for i in range(0, M, 592):
            part = nv.gemm((A[0][i:i + 592], A[1][i:i + 592], A[2]), B, fmt)
            assert bool(((part - whole[i:i + 592]).abs() <= 2 * K * 2.0 ** -24 * nA[i:i + 592, None] * nB[None]).all())


@pytest.mark.parametrize("shape,which", MIXED, ids=[n for _, n in MIXED])
def test_two_kinds_of_tiles_on_slabs(shape, which):
    M, N, K = (-(-n // 16) * 16 for n in shape)
    assert_mixed(M, N, K, which)
    assert nv.gemm_tile(M, N, K) == (256, 256)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    X, W = (torch.randn((n, K), generator=g, device="cuda") for n in (M, N))
    print(f"[case] two kinds of tiles on slabs {M}x{N}x{K}", flush=True)
    ops = [(nv.quantize_dual(t)[0], nv.quantize_dual(t, slab_rows=True)[0]) for t in (X, W)]
    plain = nv.gemm(ops[0][0], ops[1][0], shape=(M, N, K))
    for slabs in ((True, False), (False, True), (True, True)):
        assert torch.equal(nv.gemm(ops[0][slabs[0]], ops[1][slabs[1]], slabs=slabs, shape=(M, N, K)), plain), slabs
