"""MXFP4 products on the direct-to-LDS kernel whose last rows of 256 hold one row, on short contractions: the loads past the end of the contraction
stay in range there, and the bits are those of row-major operands."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_gemm_close, ofmt, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [512, 640, 768])
@pytest.mark.parametrize("M,N", [(1025, 11008), (11008, 1025)])
def test_one_row_in_the_last_tile(M, N, K):
    from paper_2505_19115_amd import binding as nv
    fmt = nv.MXFP4
    assert nv.gemm_tile(M, N, K, fmt) == (256, 256)
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    X, W = (torch.randn((n, K), generator=g, device="cuda") for n in (M, N))
    print(f"[case] MXFP4 {M}x{N}x{K}, row-major and slab operands", flush=True)
    rows = [nv.quantize(t, 1, nv.RTN, 0, fmt) for t in (X, W)]
    rows = [(q[0], q[1], torch.ones(1, device="cuda")) for q in rows]
    # (both orientations need whole blocks of rows: the operand of 11008 rows is the one that comes in slabs)
    big = 0 if M > N else 1
    slab = nv.quantize_dual((X, W)[big], fmt=fmt, slab_rows=True)[0]
    ops = list(rows)
    ops[big] = (slab[0], slab[1], rows[big][2])
    plain = nv.gemm(*rows, fmt)
    got = nv.gemm(*ops, fmt, slabs=(big == 0, big == 1), shape=(M, N, K))
    torch.cuda.synchronize()
    assert torch.equal(got, plain)
    rng = np.random.default_rng(K)
    ii, jj = rng.integers(0, M, 2000), rng.integers(0, N, 2000)
    ii[:200] = M - 1
    jj[200:400] = N - 1
    A, B = [(to_np(q[0]), to_np(q[1]), 1.0) for q in rows]
    assert_gemm_close(to_np(got)[ii, jj], oracle.gemm_nt_sample(A, B, ii, jj, ofmt(fmt)), oracle.gemm_nt_sample(A, B, ii, jj, ofmt(fmt), take_abs=True), f"{M}x{N}x{K}")
