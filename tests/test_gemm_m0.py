"""The INT8 GEMM sets M0 in assembly for its LDS-direct loads and does not tell the compiler (M0 cannot be declared
as clobbered): nothing else in these kernels may use it, which the assembly of the source shows."""
import os
import re
import subprocess

from paper_2508_03984_amd import build


def test_nothing_but_the_loads_uses_m0(tmp_path):
    asm = tmp_path / "gemm.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([build.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S",
                                                   os.path.join(build.CSRC, "oz2_int8_gemm.hip"), "-o", str(asm)])
    lines = [line.strip() for line in asm.read_text().splitlines() if not line.strip().startswith(";")]
    at = [i for i, line in enumerate(lines) if re.search(r"\bm0\b", line)]
    assert at
    for i in at:
        assert re.match(r"s_mov_b32 m0, s\d+$", lines[i]), lines[i]
        assert lines[i + 1] == "s_nop 0" and lines[i + 2].startswith("global_load_lds_dwordx4"), lines[i:i + 3]
    loads = sum(line.startswith("global_load_lds_dwordx4") for line in lines)
    assert 2 * len(at) <= loads <= 4 * len(at)
