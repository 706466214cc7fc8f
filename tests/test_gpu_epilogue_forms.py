"""Accumulation: every number of moduli has a kernel of its own; widths around its groups of four columns, destinations that
are not 16-byte aligned and a C that is read (beta), against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2508_03984_amd as oz
import synth_inputs as S
from oracle import oz2_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("N", list(range(2, 21)))
def test_each_number_of_moduli(dtype, N):
    m, n, k = 33, 258 + N % 4, 1300                  # beyond the one-launch form
    A, B = S.gemm_inputs(m, n, k, 0.5, seed=N, dtype=dtype)
    ref = O.gemm(A, B, N, is_double=dtype == np.float64)["C"].astype(np.float64)
    ld = n + 3
    C = torch.full((m, ld), 2.0, dtype=torch.from_numpy(A).dtype, device="cuda")
    out = C[:, 1:1 + n]                              # odd offset and leading dimension
    oz.matmul(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), N, out=out)
    tol = 1e-14 if dtype == np.float64 else 2.0 ** -23
    got = out.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - ref) / np.where(ref == 0, 1.0, np.abs(ref))) <= tol
    assert torch.all(C[:, 0] == 2.0) and torch.all(C[:, 1 + n:] == 2.0)
    # beta = 1 on an aligned C gives fma(1, c, C): one rounding of the sum
    D = torch.ones((m, n), dtype=C.dtype, device="cuda")
    oz.matmul(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), N, beta=1.0, out=D)
    want = (ref + 1.0).astype(dtype).astype(np.float64)
    eps = np.finfo(dtype).eps
    assert np.max(np.abs(D.cpu().numpy() - want)) <= 4 * eps * np.max(np.abs(ref) + 1.0)
