"""The work of an INT8 GEMM launch (csrc/oz2_tilemap.hpp), built for the host: its tiles and the tiles of padding cover every
entry of every plane once, and the K ranges of a slice every K tile once."""
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
using namespace oz2;
static long bad = 0;
// computed entries (in blocks of 128 x 128) exactly once, blocks of padding at most once, and by tiles within the panel
static void check(int hm, int hn, int tile, int batch, int ranges, int kt) {
    const int rows = (hm + 1) / 2 * 256, cols = (hn + 1) / 2 * 256, W = cols / 128;
    // 1: the last row / column of the last block, 128: all of it
    for (int inside : {1, 128}) {
        const GemmGrid g = make_gemm_grid(rows, cols, 128 * (hm - 1) + inside, 128 * (hn - 1) + inside, tile, batch, ranges, kt);
        const int planes = batch * ranges;
        std::vector<int> done(planes * (rows / 128) * W, 0);
        auto cover = [&](const GemmItem &it, bool padding) {
            if (it.plane < 0 || it.plane >= planes || it.s != it.plane % batch) { ++bad; return; }
            if (it.tr < 0 || it.tc < 0 || (it.tr + 1) * tile > rows || (it.tc + 1) * tile > cols) { ++bad; return; }
            for (int r = 0; r < tile / 128; ++r)
                for (int c = 0; c < tile / 128; ++c) {
                    const int br = it.tr * tile / 128 + r, bc = it.tc * tile / 128 + c;
                    if (padding && br < hm && bc < hn) ++bad;
                    ++done[(it.plane * (rows / 128) + br) * W + bc];
                }
        };
        for (int id = 0; id < g.map.total; ++id) {
            const GemmItem it = map_item(g, id);
            const int range = it.plane / batch;
            int first = 0;
            for (int r = 0; r < range; ++r) first += 2 * (kt / 2 / ranges + (r < kt / 2 % ranges ? 1 : 0));
            if (it.kt < 2 || it.kb != first || it.kt != 2 * (kt / 2 / ranges + (range < kt / 2 % ranges ? 1 : 0))) ++bad;
            if (range == ranges - 1 && it.kb + it.kt != kt) ++bad;
            cover(it, false);
        }
        for (int j = 0; j < g.padding; ++j) {
            const GemmItem it = padding_item(g, j);
            if (it.plane >= batch) ++bad;                                  // of the first range only
            cover(it, true);
        }
        for (int p = 0; p < planes; ++p)
            for (int r = 0; r < rows / 128; ++r)
                for (int c = 0; c < W; ++c) {
                    const int want = p < batch || (r < hm && c < hn) ? 1 : -1;   // padding of later ranges: at most once
                    const int got = done[(p * (rows / 128) + r) * W + c];
                    if (want == 1 ? got != 1 : got > 1) ++bad;
                }
    }
}
int main(int argc, char **argv) {
    const int lo = std::atoi(argv[1]), hi = std::atoi(argv[2]);
    for (int m = lo; m < hi; ++m)
        for (int n = 1; n < 36; ++n)
            for (int b : {1, 6, 15})
                for (int ranges : {1, 2, 7}) {
                    check(m, n, 256, b, ranges, 14 + m % 5 * 2);
                    check(m, n, 128, b, ranges, 14 + n % 7 * 2);
                }
    std::printf("bad=%ld\n", bad);
    return bad != 0;
}
"""


@pytest.mark.parametrize("lo,hi", [(1, 8), (8, 14), (31, 34)])
def test_every_block_once(tmp_path, lo, hi):
    src = tmp_path / "grid_main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "grid"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fsanitize=undefined", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe), str(lo), str(hi)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout + out.stderr[-500:]


PLAN = r"""
#include <cstdio>
#include "oz2_plan.hpp"
using namespace oz2;
int main() {
    long bad = 0, several = 0;
    const int64_t sizes[] = {1, 100, 128, 129, 256, 257, 300, 512, 600, 777, 1024, 1280, 1536, 2048, 3000, 5000, 16384};
    const int64_t ks[] = {1, 128, 1000, 1536, 2048, 3000, 4096, 8192, 20000, 40000, 131072, 131073, 200000};
    for (int64_t m : sizes)
        for (int64_t n : sizes)
            for (int64_t k : ks)
                for (int N = 2; N <= 20; N += 3) {
                    const Layout L = make_layout(m, n, k, N, true);
                    const int64_t kt = L.Kp / kBlockK;
                    if (L.ranges < 1 || L.ranges > kMaxRanges || L.prod_ranges != (size_t)(L.ranges - 1) * N * L.Mp * L.Np) ++bad;
                    if (make_layout(m, n, k, N, false).ranges != 1) ++bad;
                    if (L.ranges == 1) continue;
                    ++several;
                    if (kt / L.ranges < 12 || k > OZ2_MAX_K) ++bad;
                    if (launch_panels(L.Mp, L.Np, L.Kp).count != 1 || launch_k_len(L.Kp, N, launch_panels(L.Mp, L.Np, L.Kp)) != L.Kp) ++bad;
                    const GemmPlan p = gemm_plan(m, n, N, kt, true);       // what the launch works out
                    if (p.ranges != L.ranges || p.tile == GemmTile::kTwoPerUnit) ++bad;
                    if (p.tile == GemmTile::kOnePerUnit && blocks_of_128(m, n) * N * p.ranges > 256) ++bad;
                    if (L.prod_ranges > (size_t)448 * kMaxRanges * 65536) ++bad;
                }
    std::printf("bad=%ld %d\n", bad, several > 500);
    return bad != 0;
}
"""


def test_plans_of_k_ranges(tmp_path):
    src = tmp_path / "plan_main.cpp"
    src.write_text(PLAN)
    exe = tmp_path / "plan"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0 1", out.stdout + out.stderr[-500:]


LINES = r"""
#include <cstdio>
#include "oz2_plan.hpp"
using namespace oz2;
int main() {
    long m, n, k; int N;
    while (std::scanf("%ld %ld %ld %d", &m, &n, &k, &N) == 4) std::printf("%d\n", make_layout(m, n, k, N, true).ranges);
}
"""


def test_large_tiles_of_middle_contractions(tmp_path):
    """Ranges of large tiles only where they are faster than one of small tiles, which have a unit each or two share one."""
    cases = {(244, 386, 4623, 18): 1, (990, 189, 6626, 10): 1, (181, 404, 6807, 18): 1, (459, 696, 5323, 6): 1, (191, 390, 7676, 12): 9,   # a unit each
             (1012, 494, 3398, 12): 1, (1637, 618, 4286, 5): 1, (133, 1163, 4378, 18): 2,                             # two share one, k < 4480
             (967, 1484, 7032, 5): 2, (1337, 194, 5656, 16): 2, (787, 578, 6979, 9): 2,                               # ... and beyond
             (574, 264, 9904, 10): 3, (716, 202, 12328, 18): 4, (849, 1104, 6219, 16): 2,                             # 8192 and beyond; large tiles anyway
             (31, 42, 2611, 11): 3, (18, 1701, 2725, 9): 2}                                                           # ranges of small tiles
    src = tmp_path / "lines.cpp"
    src.write_text(LINES)
    exe = tmp_path / "lines"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d %d" % c for c in cases), capture_output=True, text=True)
    assert dict(zip(cases, map(int, out.stdout.split()))) == cases
