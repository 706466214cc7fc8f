"""Sizes on both sides of the limits where a call takes another kernel or another shape of one."""
import numpy as np
import pytest

import synth_inputs as S
from test_gpu_ops_panels import stored
from test_gpu_parity import assert_parity, gpu_gemm, oz  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,N,dtype", [
    (1, 1, 1, 2, np.float64),                        # one entry, one chunk of k, two moduli
    (31, 33, 128, 16, np.float64),                   # tile edges; a modulus per wavefront
    (33, 64, 129, 16, np.float64),                   # two chunks
    (100, 100, 200, 17, np.float32),                 # 17 moduli, neither factor narrow: two launches
    (100, 100, 120, 17, np.float32),                 # a second modulus for one wavefront
    (512, 500, 250, 8, np.float32),                  # 256 tiles, the most of the one-launch form
    (513, 500, 250, 8, np.float32),                  # one row more: two launches
    (64, 40, 500, 8, np.float64),                    # four chunks: the longest in a row for a wavefront
    (64, 40, 513, 7, np.float64),                    # longer: two launches
    (255, 257, 127, 20, np.float64),                 # all moduli
])
def test_products_around_the_one_launch_form(oz, oracle, m, n, k, N, dtype):
    """The smallest products run GEMMs and accumulation as one launch: every stage and C against the
    oracle, with alpha and beta too."""
    is_double = dtype == np.float64
    A, B = S.gemm_inputs(m, n, k, 1.0, seed=900 + m + k, dtype=dtype)
    assert_parity(gpu_gemm(oz, A, B, N), oracle.gemm(A, B, N, is_double=is_double), is_double)
    Cin = S.matrix(m, n, 0.5, seed=7, dtype=dtype)
    assert_parity(gpu_gemm(oz, A, B, N, 0.5, -1.25, Cin, ldc=n + 3),
                  oracle.gemm(A, B, N, 0.5, -1.25, Cin, is_double=is_double), is_double)


@pytest.mark.parametrize("m,n", [(1, 1), (33, 250), (256, 100), (300, 31)])
def test_padding_of_the_smallest_products_is_zero(oz, m, n):
    """U_s beyond m x n holds zeros, whatever the workspace held before."""
    import torch
    from paper_2508_03984_amd import binding as b
    k, N = 100, 15
    A, B = S.gemm_inputs(m, n, k, 1.0, seed=41)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    dC = torch.empty((m, n), dtype=torch.float64, device="cuda")
    ws = torch.full((oz.oz2_workspace_bytes(m, n, k, N),), 0x5A, dtype=torch.int8, device="cuda")
    oz.oz2_set_workspace(ws)
    try:
        oz.oz2_dgemm(m, n, k, 1.0, dA, k, dB, n, 0.0, dC, n, N)
        torch.cuda.synchronize()
        U = oz.stage_tensor(b.OZ2_STAGE_U).clone()
    finally:
        oz.oz2_set_workspace(None)
    assert U.shape == (N, 256 if m <= 256 else 512, 256)
    assert not U[:, m:, :].any() and not U[:, :, n:].any()


@pytest.mark.parametrize("k", [128, 129, 256, 257])
def test_short_contractions_with_several_tiles_per_workgroup(oz, oracle, k):
    """480 tiles of 256 x 256 for the persistent GEMM's workgroups, and K tiles around its pipeline: 2 (the head is
    shorter than the pipeline), 4 (one prefetching iteration, which takes the relaxed wait) and 6."""
    m, n, N = 1100, 1500, 16
    A, B = S.gemm_inputs(m, n, k, 1.0, seed=700 + k)
    assert_parity(gpu_gemm(oz, A, B, N), oracle.gemm(A, B, N), True)


@pytest.mark.parametrize("m,n,k,opA,opB", [
    (5, 3, 7, 0, 1), (5, 3, 7, 1, 0),                # rows shorter than one 8-element piece
    (37, 300, 129, 0, 0), (300, 37, 511, 1, 1),      # smallest workgroups, ragged rows and columns
    (40, 50, 1025, 0, 1), (40, 50, 1025, 1, 0),      # beyond 1024: other shapes for rows and for columns
    (30, 600, 2049, 0, 0),                           # beyond 2048: a launch per form
    (300, 700, 2048, 1, 0), (5, 3, 1500, 0, 0),      # few vectors: 4 and 2 per workgroup where many take 16
    (1500, 1111, 2900, 1, 0),                        # strips of 4 columns
    (20, 30, 4096, 1, 0), (20, 30, 4097, 1, 0),      # the longest columns, and beyond: the general column kernels
    (9, 270, 16384, 0, 1), (9, 270, 16385, 0, 1),    # the longest rows, and beyond: rows held for their shifts only
    (3, 4, 40961, 0, 1), (3, 4, 49153, 0, 1),        # ... by the largest workgroup; read twice
])
@pytest.mark.parametrize("dtype,N,accurate", [(np.float64, 16, False), (np.float32, 8, False), (np.float64, 9, True)])
def test_conversion_forms_agree(oz, m, n, k, opA, opB, dtype, N, accurate):
    """The fused conversion against the general kernels (which the oracle checks elsewhere): shifts, slices with
    their padding, and C are equal bit for bit; leading dimensions leave rows unaligned."""
    import torch
    from paper_2508_03984_amd import binding as b
    A, B = S.gemm_inputs(m, n, k, 2.0, seed=31 + k, dtype=dtype)
    A[m // 2, :] = 0.0
    B[:, n // 3] = 0.0
    is_double = dtype == np.float64
    dt = torch.float64 if is_double else torch.float32
    dA, lda = stored(A, opA, 3, dt)
    dB, ldb = stored(B, opB, 5, dt)
    fn = oz.oz2_dgemm_op if is_double else oz.oz2_sgemm_op
    got = {}
    try:
        for fused in (True, False):
            oz.oz2_set_small_conversion(fused)
            dC = torch.full((m, n), float("nan"), dtype=dt, device="cuda")
            fn(opA, opB, accurate, m, n, k, 1.0, dA, lda, dB, ldb, 0.0, dC, n, N)
            torch.cuda.synchronize()
            got[fused] = [dC] + [oz.stage_tensor(st) for st in (b.OZ2_STAGE_SHIFT_A, b.OZ2_STAGE_SHIFT_B,
                                                                b.OZ2_STAGE_RES_A, b.OZ2_STAGE_RES_B)]
    finally:
        oz.oz2_set_small_conversion(True)
    for x, y, name in zip(got[True], got[False], ("C", "tA", "tB", "residues of A", "residues of B")):
        assert torch.equal(x, y), name
    assert bool(torch.isfinite(got[True][0]).all())


@pytest.mark.parametrize("m,n,k,opA,opB", [
    (20, 30, 4096, 1, 0), (20, 30, 4097, 1, 0),      # both factors by columns: the longest that are fused, and beyond
    (9, 270, 16384, 0, 1), (9, 270, 16385, 0, 1),    # both by rows
])
@pytest.mark.parametrize("dtype,N", [(np.float64, 16), (np.float32, 8)])
def test_prepared_operands_of_both_conversions(oz, m, n, k, opA, opB, dtype, N):
    """A product of prepared operands equals the plain call bit for bit, whichever kernels converted them."""
    import torch
    A, B = S.gemm_inputs(m, n, k, 2.0, seed=61 + k, dtype=dtype)
    is_double = dtype == np.float64
    dt = torch.float64 if is_double else torch.float32
    dA, lda = stored(A, opA, 3, dt)
    dB, ldb = stored(B, opB, 5, dt)
    fn = oz.oz2_dgemm_op if is_double else oz.oz2_sgemm_op
    prepare = oz.oz2_prepare_d if is_double else oz.oz2_prepare_s
    product = oz.oz2_dgemm_prepared if is_double else oz.oz2_sgemm_prepared
    want = torch.full((m, n), float("nan"), dtype=dt, device="cuda")
    fn(opA, opB, False, m, n, k, 1.0, dA, lda, dB, ldb, 0.0, want, n, N)
    try:
        for fused in (True, False):
            oz.oz2_set_small_conversion(fused)
            left, right = prepare(0, opA, m, k, dA, lda, N), prepare(1, opB, n, k, dB, ldb, N)
            got = torch.full((m, n), float("nan"), dtype=dt, device="cuda")
            product(left, right, 1.0, 0.0, got, n)
            torch.cuda.synchronize()
            assert torch.equal(got, want), fused
            left.free(); right.free()
    finally:
        oz.oz2_set_small_conversion(True)
