"""The INT8 GEMM by 4 wavefronts: numbers of K tiles around what its stream of K tiles needs, one to several tiles per workgroup, K ranges of
different lengths, and the largest sums; exact, against the int32 sums of the other kernels."""
import pytest
import torch

import paper_2508_03984_amd as oz
from paper_2508_03984_amd import binding as b

pytestmark = pytest.mark.gpu


def residues_and_product(A, B, N):
    """U_s of the default form, the same from the int32 sums, and both products."""
    out = []
    try:
        for int32 in (False, True):
            oz.oz2_set_int32_products(int32)
            C = oz.matmul(A, B, N)
            torch.cuda.synchronize()
            if int32:
                p = torch.tensor(oz.oz2_constants(N)["p"][:N].tolist(), dtype=torch.int32, device="cuda").view(N, 1, 1)
                U = torch.remainder(oz.stage_tensor(b.OZ2_STAGE_PROD), p).to(torch.uint8)
            else:
                U = oz.stage_tensor(b.OZ2_STAGE_U).clone()
            out += [U, C]
    finally:
        oz.oz2_set_int32_products(False)
    return out


# tiles: 340 (a second one for 84 workgroups), 320, 768 (three each), 1000 (ragged, four), and for short contractions 2112 and 2304
@pytest.mark.parametrize("m,n,N,k", [(1000, 1050, 17, k) for k in (768, 890, 1100)] + [(1024, 1279, 16, k) for k in (700, 1024)] +
                         [(2048, 2048, 12, 1100), (2550, 2500, 10, 768), (2550, 2500, 10, 2000)] +
                         [(3000, 2700, 16, k) for k in (321, 512)] + [(3072, 3072, 16, k) for k in (384, 640)])
def test_numbers_of_k_tiles(m, n, N, k):
    gen = torch.Generator(device="cuda").manual_seed(k)
    A = torch.rand((m, k), dtype=torch.float64, device="cuda", generator=gen) - 0.5
    B = torch.rand((k, n), dtype=torch.float64, device="cuda", generator=gen) - 0.5
    for _ in range(3):                                         # with operands in the caches, too
        U, C, U32, C32 = residues_and_product(A, B, N)
        assert torch.equal(U, U32) and torch.equal(C, C32)


@pytest.mark.parametrize("m,n,k,N", [(1024, 1024, 8192, 15),     # one tile per workgroup, a long contraction
                                     (700, 600, 30000, 16),      # K ranges of different lengths, several per workgroup
                                     (600, 700, 65536, 7)])
def test_long_contractions(m, n, k, N):
    gen = torch.Generator(device="cuda").manual_seed(k)
    A = torch.rand((m, k), dtype=torch.float32, device="cuda", generator=gen) - 0.5
    B = torch.rand((k, n), dtype=torch.float32, device="cuda", generator=gen) - 0.5
    U, C, U32, C32 = residues_and_product(A, B, N)
    assert torch.equal(U, U32) and torch.equal(C, C32)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_the_largest_sums(sign):
    """All residues modulo 256 are -128, whatever the sign (-128 = 128 there): sums of 2^30, the largest that any slice can have."""
    m, n, k, N = 1024, 1024, 65536, 16
    A = torch.ones((m, k), dtype=torch.float64, device="cuda")
    oz.matmul(A[:256], A[:256].t(), N)
    torch.cuda.synchronize()
    f = int(oz.stage_tensor(b.OZ2_STAGE_SHIFT_A)[0])            # the scaled integers are below 2^(f + 1)
    A *= 1.0 + 2.0 ** (7 - f)                                   # 2^f + 128
    B = sign * A[:n].t()
    U, C, U32, C32 = residues_and_product(A, B, N)
    oz.matmul(A, B, N)
    torch.cuda.synchronize()
    assert bool((oz.stage_tensor(b.OZ2_STAGE_RES_A)[0] == -128).all())
    assert torch.equal(U, U32) and torch.equal(C, C32)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("p", [255, 253])
def test_the_largest_sums_of_an_odd_modulus(sign, p):
    """All residues of A are (p - 1) / 2 modulo p and those of B the same or the opposite: for p = 255 sums of +-127^2 65536, next to
    which a sum that left its side of zero would have another residue."""
    m, n, k, N = 1024, 1024, 65536, 14
    s = oz.oz2_constants(N)["p"].tolist().index(p)
    A = torch.ones((m, k), dtype=torch.float64, device="cuda")
    oz.matmul(A[:256], A[:256].t(), N)
    torch.cuda.synchronize()
    f = int(oz.stage_tensor(b.OZ2_STAGE_SHIFT_A)[0])            # the scaled integers are below 2^(f + 1)
    assert 8 < f <= 52
    half = (p - 1) // 2
    A *= 1.0 + (half - 2 ** f) % p * 2.0 ** -f                  # 2^f + r = half (mod p)
    B = sign * A[:n].t()
    U, C, U32, C32 = residues_and_product(A, B, N)
    assert bool((oz.stage_tensor(b.OZ2_STAGE_PROD)[s] == sign * half * half * k).all())
    oz.matmul(A, B, N)
    torch.cuda.synchronize()
    assert bool((oz.stage_tensor(b.OZ2_STAGE_RES_A)[s] == half).all())
    assert bool((oz.stage_tensor(b.OZ2_STAGE_RES_B)[s] == sign * half).all())
    assert bool((U[s] == sign * half * half * k % p).all())
    assert torch.equal(U, U32) and torch.equal(C, C32)
