"""The map from workgroup ids to output tiles of the INT8 GEMM (csrc/oz2_tilemap.hpp), built for the host: every
launch covers every tile of every slice exactly once."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_03984_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "oz2_tilemap.hpp"
int main(int argc, char **argv) {
    const int lo = std::atoi(argv[1]), hi = std::atoi(argv[2]);
    const int batches[] = {1, 2, 7, 16, 20};
    long bad = 0;
    for (int m = lo; m < hi; ++m)
        for (int n = 1; n < 50; ++n)
            for (int b : batches) {
                const int total = m * n * b;
                std::vector<char> seen(total, 0);
                const oz2::TileMap t = oz2::make_tile_map(m, n, total);
                for (int id = 0; id < total; ++id) {
                    int s, r, c;
                    oz2::map_tile(t, id, s, r, c);
                    const bool in = s >= 0 && s < b && r >= 0 && r < m && c >= 0 && c < n;
                    if (!in || seen[(s * m + r) * n + c]) { ++bad; break; }
                    seen[(s * m + r) * n + c] = 1;
                }
            }
    // the divisions of the map
    for (int64_t d = 1; d < (1ll << 31); d += d < 4096 ? 1 : d / 3) {
        const oz2::Divisor by = oz2::make_divisor((int)d);
        for (int64_t q : {(int64_t)0, (int64_t)1, (int64_t)2, 0x7fffffff / d / 2, 0x7fffffff / d - 1, 0x7fffffff / d})
            for (int64_t x : {q * d - 1, q * d, q * d + 1, q * d + d - 1, (int64_t)0x7fffffff})
                if (x >= 0 && x <= 0x7fffffff && oz2::divide((int)x, by) != x / d) ++bad;
    }
    std::printf("bad=%ld\n", bad);
    return bad != 0;
}
"""


@pytest.mark.parametrize("lo,hi", [(1, 18), (18, 34), (63, 66)])
def test_every_tile_once(tmp_path, lo, hi):
    src = tmp_path / "tilemap_main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "tilemap"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe), str(lo), str(hi)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout
