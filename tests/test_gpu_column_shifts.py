"""The shifts of columns from one read: tiles of a column whose maxima lie any number of binades below the column's, columns whose
sum of squares is close to a threshold of the shift, against the oracle."""
import math

import numpy as np
import pytest
import torch

import paper_2508_03984_amd as oz
from oracle import constants as K
from paper_2508_03984_amd import binding as b

pytestmark = pytest.mark.gpu

TILE = 128                                               # rows of a column per workgroup


def column_shifts(B, N):
    k, n = B.shape
    is_double = B.dtype == np.float64
    dt = torch.float64 if is_double else torch.float32
    A = torch.ones((2, k), dtype=dt, device="cuda")
    wide = torch.full((k, n + 3), 7.0, dtype=dt, device="cuda")         # what lies beyond a row is not read as part of it
    wide[:, :n] = torch.from_numpy(B).cuda()
    C = torch.empty((2, n), dtype=dt, device="cuda")
    (oz.oz2_dgemm if is_double else oz.oz2_sgemm)(2, n, k, 1.0, A, k, wide, n + 3, 0.0, C, n, N)
    torch.cuda.synchronize()
    return oz.stage_tensor(b.OZ2_STAGE_SHIFT_B).cpu().numpy()


@pytest.mark.parametrize("dtype,N", [(np.float64, 15), (np.float32, 8)])
@pytest.mark.parametrize("k,n", [(4097, 1), (4352, 63), (4353, 64), (5000, 65), (9001, 130), (16385, 70), (40001, 70), (65537, 9),
                                 (270000, 5)])
def test_tiles_of_any_scale(oracle, k, n, dtype, N):
    rng = np.random.default_rng(k + n)
    B = (rng.random((k, n)) - 0.5) * np.exp(0.5 * rng.standard_normal((k, n)))
    tiles = -(-k // TILE)
    scale = np.ldexp(1.0, -rng.integers(0, 9, (tiles, n)) * rng.integers(0, 5, n))     # some columns of one scale
    scale[rng.random((tiles, n)) < 0.1] = 0.0            # tiles of zeros
    B *= np.repeat(scale, TILE, axis=0)[:k]
    B[:, n // 2] *= 2.0 ** (-1060 if dtype == np.float64 else -140)                    # subnormal numbers
    if n > 2:
        B[:, 1] = 0.0
        B[:, 0] = 0.0
        B[k - 1, 0] = -3.0                               # one number, in the last row
    B = B.astype(dtype)
    want, _, _ = oracle.shifts(B.astype(np.float64), 1, K.constants(N).Pfast)
    assert np.array_equal(column_shifts(B, N), want)


@pytest.mark.parametrize("dtype,N", [(np.float64, 16), (np.float32, 8)])
@pytest.mark.parametrize("below", [2, 3, 5, 8])
def test_sums_at_a_threshold(oracle, below, dtype, N):
    """The first tile alone has the maximum; the others lie `below` binades lower, so that from 3 on only an interval of
    theirs is stored.  The first tile's sum puts the whole one up to 32 steps below or above a threshold."""
    k, n = 4500, 64
    Pfast = K.constants(N).Pfast
    rng = np.random.default_rng(below)
    B = np.zeros((k, n))
    B[TILE:] = np.ldexp(0.5 + 0.5 * rng.random((k - TILE, n)), 1 - below).astype(dtype)
    B[np.arange(k) % 8 != 0] = 0.0
    rest = np.square(np.ceil(B * 2.0 ** 15)).sum(axis=0)
    # the shift falls by one where 0.51 log2(T 2^-30) crosses Pfast - j; here between 2^36.5 and 2^38.5
    j = math.floor(Pfast - 0.51 * 6.5)
    theta = math.floor(2.0 ** (30 + (Pfast - j) / 0.51))
    step = max(1, int(0.1 * math.sqrt(TILE * rest.max()) / 2))
    for c in range(n):
        left = theta - int(rest[c]) + (c - n // 2) * step
        assert left > 2 ** 32
        i = 0
        while left > 0:                                  # a sum of squares of q <= 65535
            q = min(65535, math.isqrt(left))
            B[i, c] = math.ldexp(q, -15)
            left -= q * q
            i += 1
        assert i <= TILE
    B = B.astype(dtype)
    want, e, _ = oracle.shifts(B.astype(np.float64), 1, Pfast)
    assert (e == 0).all() and len(set(want)) == 2        # both sides of the threshold
    assert np.array_equal(column_shifts(B, N), want)


def at_a_threshold(k, n, below, live, dtype, N):
    """Columns with sums up to n / 2 steps below or above a threshold: every `live`-th tile lies `below` binades under the first, the others
    one or two, which are known exactly and not read again."""
    Pfast = K.constants(N).Pfast
    rng = np.random.default_rng(k)
    tile = np.arange(k) // TILE
    down = np.where(tile % live == 0, below, 1 + tile % 2)
    sparse = np.arange(k) % 97 == 5
    B = np.ldexp(0.5 + 0.5 * rng.random((k, n)), 1 - down[:, None]).astype(dtype).astype(np.float64)
    B[~sparse] = 0.0
    B[(tile % live != 0) & (np.arange(k) % (97 * 64) != 5)] = 0.0
    B[:TILE] = 0.0
    rest = np.square(np.ceil(B * 2.0 ** 15)).sum(axis=0)
    far = np.square(np.ceil(B[tile % live == 0] * 2.0 ** 15)).sum(axis=0)
    j = math.floor(Pfast - 0.51 * 6.5)
    theta = math.floor(2.0 ** (30 + (Pfast - j) / 0.51))
    step = max(1, int(0.1 * math.sqrt(TILE * far.max()) / n))
    for c in range(n):
        left = theta - int(rest[c]) + (c - n // 2) * step
        assert left > 2 ** 32
        i = 0
        while left > 0:
            q = min(65535, math.isqrt(left))
            B[i, c] = math.ldexp(q, -15)
            left -= q * q
            i += 1
        assert i <= TILE
    return B.astype(dtype)


@pytest.mark.parametrize("dtype,N", [(np.float64, 16), (np.float32, 8)])
@pytest.mark.parametrize("k,n,below,live", [(17000, 9, 4, 1), (40000, 70, 5, 3), (65536, 3, 8, 2), (65537, 5, 6, 1), (130000, 70, 7, 5),
                                            (300001, 3, 8, 1)])
def test_long_columns_at_a_threshold(oracle, k, n, below, live, dtype, N):
    """The second read by the workgroup that finds it necessary, for 16 columns and for 4, and from 65537 rows on by a launch of its own."""
    B = at_a_threshold(k, n, below, live, dtype, N)
    want, e, _ = oracle.shifts(B.astype(np.float64), 1, K.constants(N).Pfast)
    assert (e == 0).all() and len(set(want)) == 2
    for _ in range(3):
        assert np.array_equal(column_shifts(B, N), want)


@pytest.mark.parametrize("n,every", [(4200, 1), (4200, 16), (330, 1), (1000, 200)])
def test_strips_of_a_second_read(oracle, n, every):
    """More strips of 16 columns to read again than workgroups of that launch, fewer, and a few among others: one column near a threshold,
    scaled by powers of two and with either sign, in every `every`-th place, and columns of ones."""
    k, N = 65600, 8
    column = at_a_threshold(k, 1, 6, 1, np.float32, N)
    ones = np.ones((k, 1), np.float32)
    shift, one = (oracle.shifts(x.astype(np.float64), 1, K.constants(N).Pfast)[0][0] for x in (column, ones))
    place = torch.arange(n, device="cuda")
    B = torch.where(place % every == 0, torch.from_numpy(column).cuda(), torch.from_numpy(ones).cuda())
    B *= torch.ldexp(torch.where(place % 2 == 0, 1.0, -1.0).cuda(), place % 7 - 3)
    want = torch.where(place % every == 0, int(shift), int(one)) - (place % 7 - 3)
    A = torch.ones((2, k), dtype=torch.float32, device="cuda")
    C = torch.empty((2, n), dtype=torch.float32, device="cuda")
    for _ in range(3):
        oz.oz2_sgemm(2, n, k, 1.0, A, k, B, n, 0.0, C, n, N)
        torch.cuda.synchronize()
        assert torch.equal(oz.stage_tensor(b.OZ2_STAGE_SHIFT_B).long(), want)
