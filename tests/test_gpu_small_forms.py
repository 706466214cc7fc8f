"""The smallest products: both tile sizes of the one-launch form and both sides of the line between them, its order of tiles
for wide, tall and uneven grids, and conversions that spread the groups of moduli over workgroups."""
import numpy as np
import pytest

import synth_inputs as S
from test_gpu_parity import assert_parity, gpu_gemm, oz  # noqa: F401  (fixture)
from test_launch_routes import ONE, TWO

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,N,dtype", [
    (256, 256, 256, 14, np.float64),                 # 256 tiles of 16 x 16, no padding
    (241, 255, 130, 16, np.float64),                 # the same, ragged
    (256, 240, 128, 15, np.float64),                 # 240 tiles and the padding beside them: 256 workgroups
    (255, 224, 128, 15, np.float64),                 # 224 and 16
    (272, 240, 100, 15, np.float32),                 # 255 tiles and padding rows: beyond, 32 x 32
    (16, 16, 64, 2, np.float64),                     # one tile
    (17, 15, 65, 20, np.float64),                    # two, a second modulus for four wavefronts
    (40, 300, 128, 14, np.float64),                  # wide: tiles dealt down the columns
    (300, 40, 128, 14, np.float32),                  # tall
    (64, 1000, 256, 15, np.float64),                 # wide, 32 x 32
    (1000, 64, 256, 15, np.float64),
    (300, 300, 256, 15, np.float64),                 # 100 tiles, which 8 does not divide
    (100, 90, 200, 18, np.float64),                  # four groups of moduli in 256 workgroups, operands for the INT8 GEMM
    (100, 90, 200, 15, np.float64),                  # three groups in 192
    (100, 90, 257, 18, np.float64),                  # longer vectors, fewer per workgroup: more than 256, not spread
    (260, 90, 200, 18, np.float64),                  # the same by their number
    (100, 90, 3000, 18, np.float64),                 # larger workgroups
    (128, 128, 512, 6, np.float32),                  # two groups, the second of one modulus
    (128, 128, 512, 5, np.float32),                  # one
])
def test_smallest_products(oz, oracle, m, n, k, N, dtype):
    is_double = dtype == np.float64
    A, B = S.gemm_inputs(m, n, k, 1.0, seed=500 + m + n, dtype=dtype)
    assert_parity(gpu_gemm(oz, A, B, N), oracle.gemm(A, B, N, is_double=is_double), is_double)
    Cin = S.matrix(m, n, 0.5, seed=8, dtype=dtype)
    assert_parity(gpu_gemm(oz, A, B, N, -1.0, 0.75, Cin, ldc=n + 1),
                  oracle.gemm(A, B, N, -1.0, 0.75, Cin, is_double=is_double), is_double)


@pytest.mark.parametrize("t,m,n,k,N", TWO + ONE)
def test_one_launch_and_two_give_the_same_bits(oz, t, m, n, k, N):
    """Prepared operands take the one-launch form where a call that converts its factors may take two launches: C, with and
    without a C that is read, is equal, and the padding of U_s is zero in both forms of the calls."""
    import torch
    from paper_2508_03984_amd import binding as b
    dtype = torch.float64 if t == "d" else torch.float32
    A, B = (torch.from_numpy(x).cuda() for x in S.gemm_inputs(m, n, k, 1.0, seed=m + k, dtype=np.float64 if t == "d" else np.float32))
    prepare, product = (oz.oz2_prepare_d, oz.oz2_dgemm_prepared) if t == "d" else (oz.oz2_prepare_s, oz.oz2_sgemm_prepared)
    left, right = prepare(0, 0, m, k, A, k, N), prepare(1, 0, n, k, B, n, N)
    try:
        for alpha, beta in ((1.0, 0.0), (-0.5, 1.25)):
            plain, one = (torch.full((m, n), 3.0, dtype=dtype, device="cuda") for _ in range(2))
            oz.matmul(A, B, N, alpha=alpha, beta=beta, out=plain)
            torch.cuda.synchronize()
            U = oz.stage_tensor(b.OZ2_STAGE_U)
            assert not U[:, m:, :].any() and not U[:, :, n:].any()
            product(left, right, alpha, beta, one, n)
            torch.cuda.synchronize()
            assert torch.equal(plain, one), (alpha, beta)
    finally:
        left.free()
        right.free()


@pytest.mark.parametrize("m,n,k,N,dtype", [
    (100, 90, 200, 18, np.float64),                  # 64 workgroups x 4 groups of moduli, the most that are spread
    (100, 90, 200, 15, np.float64),                  # x 3
    (100, 90, 257, 18, np.float64),                  # beyond: 128 x 4
    (260, 90, 200, 18, np.float64),                  # beyond: 96 x 4
    (100, 90, 200, 20, np.float32),                  # one reduction round or two, as the type asks
    (7, 250, 129, 16, np.float64),                   # the last group of one modulus
])
def test_spread_groups_of_moduli_convert_alike(oz, m, n, k, N, dtype):
    """Conversions whose groups of moduli have workgroups of their own, and those just beyond, against the general kernels:
    shifts, slices with their padding, and C are equal bit for bit."""
    import torch
    from paper_2508_03984_amd import binding as b
    A, B = (torch.from_numpy(x).cuda() for x in S.gemm_inputs(m, n, k, 2.0, seed=77, dtype=dtype))
    A[m // 2, :] = 0.0
    got = {}
    try:
        for fused in (True, False):
            oz.oz2_set_small_conversion(fused)
            C = oz.matmul(A, B, N)
            torch.cuda.synchronize()
            got[fused] = [C.clone()] + [oz.stage_tensor(st).clone() for st in (b.OZ2_STAGE_SHIFT_A, b.OZ2_STAGE_SHIFT_B,
                                                                               b.OZ2_STAGE_RES_A, b.OZ2_STAGE_RES_B)]
    finally:
        oz.oz2_set_small_conversion(True)
    for x, y, name in zip(got[True], got[False], ("C", "tA", "tB", "residues of A", "residues of B")):
        assert torch.equal(x, y), name
