"""The accumulation of int32 sums takes the moduli in groups of 8, 4, 2 and 1 and fewer wavefronts where the planes are larger
than the memory-side cache: for every number of moduli it gives the bits of the accumulation of residues."""
import pytest
import torch

import paper_2508_03984_amd as oz

pytestmark = pytest.mark.gpu

CASES = [(67, 259, N) for N in range(2, 21)] + [(2300, 2301, 12), (2300, 2301, 13), (4100, 4099, 4)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n,N", CASES)
def test_int32_sums_give_the_bits_of_residues(m, n, N, dtype):
    gen = torch.Generator(device="cuda").manual_seed(N)
    k = 300
    A = torch.rand((m, k), dtype=dtype, device="cuda", generator=gen) - 0.5
    B = torch.rand((k, n), dtype=dtype, device="cuda", generator=gen) - 0.5
    for beta in (0.0, -0.75):
        C = torch.rand((m, n), dtype=dtype, device="cuda", generator=gen)
        got = {}
        try:
            for int32 in (False, True):
                oz.oz2_set_int32_products(int32)
                got[int32] = C.clone()
                oz.matmul(A, B, N, beta=beta, out=got[int32])
                torch.cuda.synchronize()
        finally:
            oz.oz2_set_int32_products(False)
        assert torch.equal(got[True], got[False]), beta
        assert bool(torch.isfinite(got[True]).all())
