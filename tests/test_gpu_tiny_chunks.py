"""The one-launch form of the smallest products: every number of chunks of k that a wavefront has (fewer than are requested at once, as
many, more; one modulus or two), in both tile sizes, against the separate launches on int32 sums."""
import pytest
import torch

import paper_2508_03984_amd as oz

pytestmark = pytest.mark.gpu

CASES = ([(100, 90, k, N) for k, N in ((1, 15), (129, 16), (256, 17), (200, 20), (300, 14), (384, 16), (400, 3), (512, 14), (512, 9))] +
         [(400, 420, k, N) for k, N in ((128, 15), (100, 20), (256, 15), (257, 10), (500, 8), (512, 5), (256, 2))])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n,k,N", CASES)
def test_numbers_of_chunks(m, n, k, N, dtype):
    gen = torch.Generator(device="cuda").manual_seed(k + N)
    A = torch.rand((m, k), dtype=dtype, device="cuda", generator=gen) - 0.5
    B = torch.rand((k, n), dtype=dtype, device="cuda", generator=gen) - 0.5
    f64 = dtype == torch.float64
    left = (oz.oz2_prepare_d if f64 else oz.oz2_prepare_s)(0, 0, m, k, A, k, N)
    right = (oz.oz2_prepare_d if f64 else oz.oz2_prepare_s)(1, 0, n, k, B, n, N)
    product = oz.oz2_dgemm_prepared if f64 else oz.oz2_sgemm_prepared
    try:
        for alpha, beta in ((1.0, 0.0), (-0.5, 1.25)):
            got = {}
            for int32 in (False, True):
                oz.oz2_set_int32_products(int32)
                got[int32] = torch.full((m, n), 3.0, dtype=dtype, device="cuda")
                product(left, right, alpha, beta, got[int32], n)
                torch.cuda.synchronize()
            assert torch.equal(got[False], got[True]), (alpha, beta)
    finally:
        oz.oz2_set_int32_products(False)
        left.free()
        right.free()
