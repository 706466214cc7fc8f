"""The INT8 GEMM by 4 wavefronts (csrc/oz2_wide_gemm.hip): what its assembly counts on, read from the assembly of its source, and the
reduction of sums that start at -2^30."""
import os
import re
import subprocess

import pytest

from paper_2508_03984_amd import build

LOADS, STORES = 8, 16                                          # of a wavefront per K tile and per tile


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    asm = tmp_path_factory.mktemp("wide") / "wide.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([build.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S",
                                                   os.path.join(build.CSRC, "oz2_wide_gemm.hip"), "-o", str(asm)])
    out, cur = {}, None
    for line in asm.read_text().splitlines():
        m = re.match(r"(_ZN\S*k_wide_gemmILb([01])E\S*):", line)
        if m:
            cur = out.setdefault(m.group(2) == "1", [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None:
            cur.append(line.strip())
    assert set(out) == {False, True}
    return out


@pytest.mark.parametrize("fold", [False, True])
def test_only_the_assembly_uses_accumulators_and_m0(kernels, fold):
    """AGPRs appear in the MFMAs and in the reads of the reduction, each accumulator read once per tile; no scratch."""
    lines = [l for l in kernels[fold] if not l.startswith(";")]
    reads = []
    for line in lines:
        if re.search(r"\ba(\d+|\[)", line):
            if line.startswith("v_accvgpr_read_b32"):
                reads.append(int(re.search(r"a\[?(0x[0-9a-f]+|\d+)", line).group(1), 0))
            else:
                assert re.match(r"v_mfma_i32_16x16x64_i8 a\[\w+:\w+\], v\[\d+:\d+\], v\[\d+:\d+\], (a\[\w+:\w+\]|-2\.0)$", line), line
        assert "scratch_" not in line and "accvgpr_write" not in line, line
    assert sorted(reads) == sorted(2 * list(range(256)))       # a tile with another one behind it, and the last one
    for i, line in enumerate(lines):
        if re.search(r"\bm0\b", line):
            assert re.match(r"s_mov_b32 m0, s\d+$", line) and lines[i + 1] == "s_nop 0", line
            assert lines[i + 2].startswith("global_load_lds_dwordx4"), lines[i:i + 3]
    loads = sum(l.startswith("global_load_lds_dwordx4") for l in lines)
    assert loads == 4 * sum("m0" in l for l in lines)          # M0 serves four loads


def test_stores_that_the_relaxed_waits_pass(kernels):
    """All 16 stores of a tile stand between the barrier of its last K tile and that of the next one's first, with the 8 loads of a K tile;
    the last four K tiles request one each and store nothing, and no other loads are counted."""
    lines = [l for l in kernels[False] if not l.startswith(";")]
    assert not any(re.match(r"(global|flat|buffer)_load_(dword|ubyte|ushort)", l) for l in lines)
    waits = {int(w) for l in lines for w in re.findall(r"vmcnt\((\d+)\)", l)}
    assert waits <= {0, LOADS, 2 * LOADS, 3 * LOADS, 2 * LOADS + STORES}
    parts, cur = [], []
    for line in lines:
        cur.append(line)
        if line == "s_barrier":
            parts.append(cur)
            cur = []
    opening = [i for i, part in enumerate(parts) if any(l.endswith("-2.0") for l in part)]
    assert len(opening) == 2                                   # of a workgroup's first tile, and of each following one

    def count(part, what):
        return sum(l.startswith(what) for l in part)

    for i in range(opening[1] - 4, opening[1] + 1):            # the last four K tiles and the next tile's first
        assert count(parts[i], "global_load_lds") == LOADS and count(parts[i], "v_mfma") == 64, i
        assert count(parts[i], "global_store") == (STORES if i == opening[1] else 0), i
        if i > opening[1] - 4:                                 # in one piece
            assert not any(l.startswith((".LBB", "s_cbranch", "s_branch")) for l in parts[i]), i
    assert any("vmcnt(%d)" % (2 * LOADS + STORES) in l for l in parts[opening[1]][-4:])
    assert sum(count(part, "global_store") for part in parts) + count(cur, "global_store") == 2 * STORES


MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "oz2_bytemod.hpp"
int main() {
    long bad = 0;
    const uint32_t first = 0xc0000000u;
    for (int p = 29; p <= 256; p += p < 255 ? 2 : 1) {                 // odd ones, and 256
        const oz2::ByteMod b = oz2::make_byte_mod(p, first);
        auto check = [&](int64_t x) {
            const int64_t want = ((x % p) + p) % p;
            if ((oz2::byte_mod_word((uint32_t)((uint64_t)x + first), b) & 0xff) != (uint32_t)want) ++bad;
        };
        const int64_t top = p == 256 ? (int64_t)1 << 30 : (int64_t)127 * 127 * 65536;
        for (int64_t d = 0; d < 3000; ++d) { check(d); check(-d); check(top - d); check(-top + d); }
        uint64_t r = 12345;
        for (int i = 0; i < 200000; ++i) {
            r = r * 6364136223846793005ull + 1442695040888963407ull;
            check((int64_t)(r >> 33) % (2 * top + 1) - top);
        }
    }
    std::printf("bad=%ld\n", bad);
    return bad != 0;
}
"""


def test_reduction_of_sums_that_start_at_minus_2_30(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", build.CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0", out.stdout
