"""The contraction of a few tiles in K ranges at once: every stage and C as with one range, which the same call takes in a workspace
without room for the ranges' planes."""
import numpy as np
import pytest
import torch

import paper_2508_03984_amd as oz
import synth_inputs as S
from paper_2508_03984_amd import binding as b
from test_gpu_parity import assert_parity, gpu_gemm

pytestmark = pytest.mark.gpu


def ranges_of(m, n, k, N, is_double=True):
    """K ranges of a product, from the workspace it asks for beyond one 256 x 256 panel."""
    products = oz.oz2_workspace_bytes(m, n, k, N, is_double) - oz.oz2_workspace_min_bytes(m, n, k, N, is_double) + N * 65536
    return products // (N * (-(-m // 256) * 256) * (-(-n // 256) * 256))


# one row and column; ragged tiles of 128 x 128, 4 and 10 ranges of unequal numbers of K tiles; 20 moduli (two rounds of loads) and 2; a row
# of 256 columns and one more; tiles of 256 x 256 with 2 to 16 ranges
CASES = [(1, 1, 16384, 14), (130, 70, 13000, 15), (100, 257, 9000, 20), (257, 255, 40000, 2), (129, 513, 20000, 16),
         (500, 700, 8300, 17), (257, 1025, 33000, 6), (1270, 1020, 14400, 16)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n,k,N", CASES)
def test_ranges_give_the_bits_of_one_range(m, n, k, N, dtype):
    assert ranges_of(m, n, k, N) > 1
    gen = torch.Generator(device="cuda").manual_seed(N)
    A = torch.rand((m, k), dtype=dtype, device="cuda", generator=gen) - 0.5
    B = torch.rand((k, n), dtype=dtype, device="cuda", generator=gen) - 0.5
    C = torch.rand((m, n + 3), dtype=dtype, device="cuda", generator=gen)
    need = oz.oz2_workspace_bytes(m, n, k, N)
    got = {}
    try:
        for short in (0, 256):                                # all of it; too little for the ranges, enough for all else
            ws = torch.full((need - short,), 0x5A, dtype=torch.uint8, device="cuda")
            oz.oz2_set_workspace(ws)
            for beta in (0.0, -0.75):
                out = C.clone()
                oz.matmul(A, B, N, alpha=1.25, beta=beta, out=out[:, :n])
                torch.cuda.synchronize()
                U = oz.stage_tensor(b.OZ2_STAGE_U)
                assert bool((U[:, m:, :] == 0).all()) and bool((U[:, :, n:] == 0).all())
                got[short, beta] = out, U.clone()
    finally:
        oz.oz2_set_workspace(None)
    for beta in (0.0, -0.75):
        assert torch.equal(got[0, beta][1], got[256, beta][1])
        assert torch.equal(got[0, beta][0], got[256, beta][0])
        assert torch.equal(got[0, beta][0][:, n:], C[:, n:])   # beside the columns of C


@pytest.mark.parametrize("m,n,k,N,dtype", [(70, 130, 9000, 15, np.float64), (129, 40, 12000, 9, np.float32)])
def test_ranges_against_the_oracle(oracle, m, n, k, N, dtype):
    assert ranges_of(m, n, k, N) > 1
    A, B = S.gemm_inputs(m, n, k, 1.0, seed=k, dtype=dtype)
    oz.oz2_release()                                          # the library's own buffer, with room for the ranges
    assert_parity(gpu_gemm(oz, A, B, N), oracle.gemm(A, B, N, is_double=dtype == np.float64), dtype == np.float64)
