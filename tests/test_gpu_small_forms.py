"""The smallest products: both tile sizes of the one-launch form and both sides of the line between them, its order of tiles
for wide, tall and uneven grids, and conversions that spread the groups of moduli over workgroups."""
import numpy as np
import pytest

import synth_inputs as S
from test_gpu_parity import assert_parity, gpu_gemm, oz  # noqa: F401  (fixture)

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
    (100, 90, 3000, 18, np.float64),                 # four groups of moduli, operands for the INT8 GEMM
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
