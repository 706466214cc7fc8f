"""INT8 GEMM: numbers of K tiles around the depth of the LDS ring, in each of its tile configurations, with one and with
several tiles per workgroup of the persistent grid; exact."""
import pytest
import torch

import paper_2508_03984_amd as oz
import synth_inputs as S
from test_gpu_parity import assert_parity, gpu_gemm

pytestmark = pytest.mark.gpu

#  batch, Mp, Np: one 128 x 128 tile per compute unit at most, more of them (two of these); 256 x 256 tiles: 144, one per
#  workgroup, and 320, a second one for 64 of the 256 workgroups
CONFIGS = [(2, 256, 512), (6, 1024, 1024), (8, 1024, 1024), (9, 1024, 1024), (20, 1024, 1024)]


@pytest.mark.parametrize("kp", [128, 256, 384, 512, 640, 768, 1024, 4096, 4224])
@pytest.mark.parametrize("batch,mp,np_", CONFIGS)
def test_products_for_every_number_of_k_tiles(batch, mp, np_, kp):
    gen = torch.Generator(device="cuda").manual_seed(kp)
    A = torch.randint(-128, 128, (batch, mp, kp), dtype=torch.int8, device="cuda", generator=gen)
    B = torch.randint(-128, 128, (batch, np_, kp), dtype=torch.int8, device="cuda", generator=gen)
    C = torch.full((batch, mp, np_), 7, dtype=torch.int32, device="cuda")
    oz.oz2_int8_gemm(oz.block_slices(A), oz.block_slices(B), C, batch, mp, np_, kp)
    for s in range(batch):                                    # sums below 2^27: exact in FP64 whatever their order
        want = torch.matmul(A[s].double(), B[s].double().t().contiguous())
        assert torch.equal(C[s].double(), want), s


@pytest.mark.parametrize("k", [128, 384, 512, 640])
def test_residues_with_an_odd_number_of_tiles(oracle, k):
    """425 tiles of 256 x 256: the second tile of a workgroup starts while the stores of its first are on their way, with K
    tiles below (2), just beyond (6) and well beyond the ring's depth."""
    m, n, N = 1201, 1155, 17
    A, B = S.gemm_inputs(m, n, k, 1.0, seed=300 + k)
    assert_parity(gpu_gemm(oz, A, B, N), oracle.gemm(A, B, N), True)
