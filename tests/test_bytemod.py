"""The reduction of int32 sums to bytes in the INT8 GEMM's store phase (csrc/oz2_bytemod.hpp), built for the host:
the low byte it leaves is mod(x, p) for every modulus."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_03984_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "oz2_bytemod.hpp"
int main(int argc, char **argv) {
    long bad = 0;
    for (int a = 1; a < argc; ++a) {
        const int p = std::atoi(argv[a]);
        const oz2::ByteMod b = oz2::make_byte_mod(p);
        auto check = [&](int64_t x) {
            const unsigned want = (unsigned)(((x % p) + p) % p);
            if ((oz2::byte_mod_word((uint32_t)x + 0x80000000u, b) & 0xffu) != want && ++bad < 10)
                std::printf("p = %d x = %lld\n", p, (long long)x);
        };
        // ends of the range, the neighbourhood of 0 and of 2^16, and a walk that meets every byte value in
        // every position (the reduction sees x only through the four bytes of x + 2^31)
        for (int64_t d = 0; d < 70000; ++d) { check(INT32_MIN + d); check(INT32_MAX - d); check(d); check(-d); }
        for (int64_t x = INT32_MIN; x <= INT32_MAX; x += 4099) check(x);
        for (int hi = 0; hi < 256; ++hi)
            for (int lo = 0; lo < 256; ++lo)
                for (int s = 0; s < 24; s += 8)
                    check((int32_t)(0x80000000u + (((uint32_t)hi << 24) ^ ((uint32_t)lo << s) ^ 0x00ffffffu)));
    }
    std::printf("bad=%ld\n", bad);
    return bad != 0;
}
"""


def test_low_byte_is_the_residue_for_every_modulus(tmp_path):
    import paper_2508_03984_amd as oz
    p = [str(int(v)) for v in oz.oz2_constants(20)["p"]]
    assert len(p) == 20
    src = tmp_path / "bytemod_main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "bytemod"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)] + p, capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout
