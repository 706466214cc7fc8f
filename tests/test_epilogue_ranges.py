"""The accumulation's row ranges: a launch numbers its threads in 31 bits, so a larger C is cut into ranges of rows.  The
ranges cover every row once and fit, and the launches of a call get the parts of U, the shifts and C that belong to them
(seen on the CPU, on a stand-in for the HIP runtime: nothing is read)."""
import os
import subprocess

import pytest

from test_launch_routes import STAND_IN, run_on_stand_in

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_03984_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "oz2_plan.hpp"
#include "oz2_tilemap.hpp"
using namespace oz2;
int main() {
    long bad = 0, seen = 0;
    // a small limit, every place of every thread as the kernel works it out
    for (int64_t limit : {(int64_t)256, (int64_t)1024})
        for (int64_t n = 1; n < 1100; n += n < 40 ? 1 : 97)
            for (int64_t m = 1; m < 40; ++m) {
                const int64_t groups = epilogue_groups(n), rows = epilogue_rows(groups, limit);
                if (rows < 1) { bad += groups <= limit; continue; }
                const Divisor by = make_divisor((int)groups);
                int64_t next = 0, places = 0;
                for (int64_t r = 0; r < m; r += rows) {
                    const int64_t count = rows < m - r ? rows : m - r;
                    const int64_t threads = (count * groups + kEpilogueThreads - 1) / kEpilogueThreads * kEpilogueThreads;
                    if (threads > limit) ++bad;
                    for (int64_t t = 0; t < threads; ++t) {
                        const int row = divide((int)t, by);
                        if (row >= count) continue;
                        if ((r + row) * groups + (t - row * groups) != next++) ++bad;
                        ++places;
                    }
                }
                bad += places != m * groups;
                ++seen;
            }
    // the limit of the library: the last thread of a launch is below 2^31
    for (int64_t groups = 1; groups <= 0x3fffffff; groups = groups < 64 ? groups + 1 : groups * 3 / 2 + 1) {
        const int64_t rows = epilogue_rows(groups);
        const int64_t threads = (rows * groups + kEpilogueThreads - 1) / kEpilogueThreads * kEpilogueThreads;
        if (rows < 1 || threads > ((int64_t)1 << 31) - 1 || (rows + 1) * groups <= kEpilogueMaxThreads) ++bad;
    }
    if (epilogue_rows(0x40000000) != 0) ++bad;
    std::printf("bad=%ld\n", bad);
    return bad != 0 || seen < 1000;
}
"""

# The stand-in also writes down what the accumulation's launches get: the grid, and of the arguments
# (U, plane, Np, m, n, tA, tB, constants, alpha, beta, C, ldc, groups, divisor) U, m, tA, tB, C and the groups.
RECORD = r"""
static long long epi[64][7]; static int n_epi;
static void record(const char *name, dim3 g, void **a)
{ if (!strstr(name, "k_epilogue") || n_epi >= 64) return;
  long long *e = epi[n_epi++];
  e[0] = g.x; e[1] = *(long long *)a[0]; e[2] = *(long long *)a[3]; e[3] = *(long long *)a[5]; e[4] = *(long long *)a[6];
  e[5] = *(long long *)a[10]; e[6] = *(int *)a[12]; }
int epilogues(long long *out) { memcpy(out, epi, sizeof epi); int n = n_epi; n_epi = 0; return n; }
"""

CALLER = r"""
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
vp, i64 = C.c_void_p, C.c_int64
lib.oz2_sgemm.argtypes = [i64, i64, i64, C.c_float, vp, i64, vp, i64, C.c_float, vp, i64, C.c_int, vp]
lib.oz2_set_workspace.argtypes = [vp, C.c_size_t]
lib.oz2_set_int32_products.argtypes = [C.c_int]
out = {}
WS, CC = 1 << 40, 1 << 50                                     # nothing reads them
assert lib.oz2_set_workspace(WS, 1 << 44) == 0
for int32 in (0, 1):
    lib.oz2_set_int32_products(int32)
    for m, n, ldc in ((1000, 1000, 1000), (131071, 65536, 65540), (131072, 65540, 65600), (500001, 65533, 65533)):
        status = lib.oz2_sgemm(m, n, 100, 1.0, 1 << 20, 100, 1 << 30, n, 0.0, CC, ldc, 3, None)
        assert status == 0, status
        buf = (C.c_longlong * (64 * 7))()
        count = fake.epilogues(buf)
        out["%d %d %d %d" % (int32, m, n, ldc)] = [list(buf[7 * i:7 * i + 7]) for i in range(count)]
print(json.dumps(out))
"""


def test_ranges_cover_every_row_once(tmp_path):
    src = tmp_path / "ranges_main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "ranges"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    found = "{ strcat(names, known[i].name);"
    assert STAND_IN.count(found) == 1 and STAND_IN.count("int hipLaunchKernel") == 1
    stand_in = STAND_IN.replace(found, "{ record(known[i].name, g, a); strcat(names, known[i].name);")
    stand_in = stand_in.replace("int hipLaunchKernel", RECORD + "int hipLaunchKernel")
    return run_on_stand_in(tmp_path_factory.mktemp("ranges"), CALLER, stand_in)


def test_launches_get_their_ranges(launches):
    assert len(launches) == 8
    cut = 0
    for case, got in launches.items():
        int32, m, n, ldc = map(int, case.split())
        Np, groups = (n + 255) // 256 * 256, (n + 3) // 4
        assert got, case
        _, U0, _, tA0, tB0, C0, _ = got[0]
        assert C0 == 1 << 50
        row = 0
        for grid, U, count, tA, tB, c, g in got:
            assert (U, tA, tB, c) == (U0 + row * Np * (4 if int32 else 1), tA0 + 4 * row, tB0, C0 + 4 * row * ldc), case
            assert g == groups and 256 * (grid - 1) < count * groups <= 256 * grid < 1 << 31, case
            row += count
        assert row == m, case
        assert (len(got) > 1) == (m * groups > 0x7fffff00), case
        cut += len(got) > 1
    assert cut == 4
