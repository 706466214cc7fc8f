"""The byte counts that bench.py divides by its stage times, against what the kernels of each stage do."""
import pytest

import bench


def test_headline_reads_b_once_for_its_shifts():
    """16384 x 16384: A's shifts come with its residues, B's from one read; 0.40 ms for them is a rate that the memory can give."""
    n = 16384
    got = bench.bytes_of_stages(n, n, n, 16, 8)
    words = 24 * n * n // 128                                 # written, up to two thirds of it read back
    assert 8 * n * n + words <= got["shifts"] <= 8 * n * n + 2 * words + 8 * n
    assert got["shifts"] / 0.40e-3 < 1e9 * bench.HBM_PEAK_GBS
    assert got["residues"] == 2 * 8 * n * n + 2 * 16 * n * n
    assert got["int8_gemm"] == 3 * 16 * n * n and got["epilogue"] == (16 + 8) * n * n


@pytest.mark.parametrize("k,a,b", [(4096, 0, 0), (4097, 0, 1), (16384, 0, 1), (16385, 1, 1), (49152, 1, 1), (49153, 2, 1)])
def test_passes_of_the_shifts(k, a, b):
    """Reads of A and B before the residues, by the length of their vectors."""
    m, n, E = 512, 256, 4
    got = bench.bytes_of_stages(m, n, k, 8, E)["shifts"] - 4 * (m + n) - (40 * n * -(-k // 128) if b else 0)
    assert got == E * k * (a * m + b * n)


@pytest.mark.parametrize("k,a,b", [(4096, 1, 1), (5000, 1, 2), (20000, 2, 2)])
def test_passes_of_accurate_mode(k, a, b):
    """Maxima and magnitudes from one read or two, the magnitudes written and read by their product."""
    m, n, E = 512, 256, 8
    got = bench.bytes_of_stages(m, n, k, 15, E, accurate=True)["shifts"] - 4 * (m + n)
    assert got == E * k * (a * m + b * n) + 2 * (m + n) * -(-k // 128) * 128
