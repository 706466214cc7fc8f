"""The workgroup shapes of the fused conversion (fused_plan in csrc/oz2_plan.hpp), built for the host: every vector that
fused_applies accepts fits the registers of its workgroup, whatever the form, the type and the number of vectors, and
few vectors are spread over the chip."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_03984_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "oz2_plan.hpp"
using namespace oz2;
int main() {
    long bad = 0, seen = 0;
    for (int64_t Kp = kPadK; Kp <= kFusedMaxRow + 4 * kPadK; Kp += kPadK)
        for (int strips = 0; strips < 2; ++strips)
            for (int64_t vectors = kPadMN; vectors <= 65536; vectors += vectors < 8192 ? 256 : 3328)
                for (size_t element : {(size_t)4, (size_t)8}) {
                    if (!fused_applies(Kp, !strips)) continue;
                    const FusedPlan p = fused_plan(Kp, strips, vectors, element);
                    const int64_t V = (int64_t)1 << p.log_v;
                    const bool ok = V * Kp <= (int64_t)p.threads * p.pieces * 8      // the vectors fit
                                    && 8 * V <= p.threads                              // a thread holds one vector's pieces
                                    && p.log_v <= 5 && kPadMN % V == 0                 // whole workgroups, LDS arrays
                                    && ((strips ? V >= 4 : V >= 2) || vectors < 2 * V * 256)   // whole lines, see fused_plan
                                    // a workgroup for each of 256 compute units, unless it is the smallest there is
                                    && (vectors / V >= 256 || V == 1 || (p.threads == 256 && p.pieces == 1));
                    ++seen;
                    if (!ok && ++bad < 10)
                        std::printf("Kp %lld strips %d vectors %lld: %d x %d, log_v %d\n", (long long)Kp, strips,
                                    (long long)vectors, p.threads, p.pieces, p.log_v);
                }
    std::printf("bad=%ld\n", bad);
    return bad != 0 || seen < 1000;
}
"""


def test_vectors_fit_their_workgroups(tmp_path):
    src = tmp_path / "fused_plan_main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "fused_plan"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout


SPLIT = r"""
#include <cstdio>
#include "oz2_plan.hpp"
using namespace oz2;
int main() {
    long bad = 0, split = 0;
    for (int64_t Kp = kPadK; Kp <= kFusedMaxRow; Kp += kPadK)
        for (int strips = 0; strips < 2; ++strips)
            for (int64_t vectors = kPadMN; vectors <= 65536; vectors += 256)
                for (size_t element : {(size_t)4, (size_t)8}) {
                    if (!fused_applies(Kp, !strips)) continue;
                    const FusedPlan p = fused_plan(Kp, strips, vectors, element);
                    const int64_t workgroups = (vectors + ((int64_t)1 << p.log_v) - 1) >> p.log_v;
                    for (int groups = 1; groups <= 4; ++groups) {
                        const bool few = groups > 1 && workgroups * groups <= 256;
                        split += few;
                        bad += few != fused_split_applies(p, workgroups, groups);     // no launch of few is of another shape
                    }
                }
    std::printf("bad=%ld\n", bad);
    return bad != 0 || split < 100;
}
"""


def test_only_the_smallest_shape_spreads_its_moduli(tmp_path):
    """A kernel that spreads the groups of moduli exists for one shape of workgroups, and no other can have as few of them."""
    import re
    src = tmp_path / "fused_split_main.cpp"
    src.write_text(SPLIT)
    exe = tmp_path / "fused_split"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout
    # by type and number of reduction rounds: the kernels of the library that spread them
    import paper_2508_03984_amd as oz
    if not os.path.exists(oz.lib_path()):
        from paper_2508_03984_amd.build import build_library
        build_library()
    names = open(oz.lib_path(), "rb").read()
    split = set(re.findall(rb"_ZN3oz2[A-Z0-9_]*9k_convertI([df])Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb1E", names))
    assert split == {(t, b"256", b"1", r, b"0") for t in (b"d", b"f") for r in (b"1", b"2")}
