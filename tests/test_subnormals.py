"""The reduction of sums to bytes computes with subnormal binary32 numbers: the kernels that contain it run in the mode that
keeps them, also if the extra flags of the build ask for the other one."""
import json
import os
import re
import shlex
import subprocess
import sys

import pytest

from paper_2508_03984_amd import build

# Stands in for the compiler: it writes down what it is called with.
RECORDER = """#!{python}
import json, sys
json.dump(sys.argv[1:], open({out!r}, "w"))
"""


def flags_of_a_build(tmp_path, extra):
    out, fake = tmp_path / "flags.json", tmp_path / "hipcc"
    fake.write_text(RECORDER.format(python=sys.executable, out=str(out)))
    fake.chmod(0o755)
    env = dict(os.environ, HIPCC=str(fake), OZ2_EXTRA_HIPCC_FLAGS=extra)
    subprocess.check_call([sys.executable, "-m", "paper_2508_03984_amd.build"], env=env, cwd=os.path.dirname(build.HERE))
    argv = json.load(open(out))
    return argv[:argv.index("-x")]


@pytest.mark.parametrize("extra", ["", "-fgpu-flush-denormals-to-zero", "-fdenormal-fp-math=preserve-sign",
                                   "-Xclang -fdenormal-fp-math-f32=preserve-sign"])
@pytest.mark.parametrize("source,kernels", [("oz2_int8_gemm.hip", "k_int8_gemm"), ("oz2_tiny.hip", "k_tiny_product")])
def test_the_kernels_keep_subnormals(tmp_path, source, kernels, extra):
    flags = [f for f in flags_of_a_build(tmp_path, extra) if f not in ("-fPIC", "-shared")]
    assert all(f in flags for f in shlex.split(extra))
    asm = tmp_path / "kernels.s"
    subprocess.check_call([build.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S",
                                                   os.path.join(build.CSRC, source), "-o", str(asm)])
    text = asm.read_text()
    modes = re.findall(r"\.amdhsa_float_denorm_mode_32 (\d)", text)
    assert len(modes) >= 4 and text.count(".amdhsa_kernel") == len(modes) and kernels in text
    assert set(modes) == {"3"}                       # 3: kept in operands and in results
