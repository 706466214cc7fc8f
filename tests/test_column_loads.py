"""How the kernels that convert columns read their operand, from the assembly of their source."""
import os
import re
import subprocess

import pytest

from paper_2508_03984_amd import build


def kernels(tmp_path, source, name):
    asm = tmp_path / "kernels.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([build.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(asm)])
    out, cur = {}, None
    for line in asm.read_text().splitlines():
        m = re.match(r"(_ZN\S*%s\S*):" % name, line)
        if m:
            cur = out.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None:
            cur.append(line.strip())
    assert out
    return out


@pytest.mark.parametrize("source,name", [("oz2_columns.hip", "k_residues_cols"), ("oz2_small.hip", "k_small_residues")])
def test_operands_are_read_through_the_caches(tmp_path, source, name):
    """Neighbouring strips share the lines of rows that do not start at one, and the operand is read again by what follows."""
    for kernel, lines in kernels(tmp_path, source, name).items():
        loads = [l for l in lines if re.match(r"(global|flat|buffer)_load_", l)]
        assert loads, kernel
        assert not any(re.search(r"\b(nt|sc0|sc1)\b", l) for l in loads), kernel


def test_large_factors_request_all_elements_first(tmp_path):
    """8 loads of a thread in a row without a wait between them: the 8 elements of its piece."""
    for kernel, lines in kernels(tmp_path, "oz2_columns.hip", "k_residues_cols").items():
        run = best = 0
        for l in lines:
            if re.match(r"global_load_dword(x2)? ", l):
                run += 1
                best = max(best, run)
            elif "vmcnt" in l:
                run = 0
        assert best >= 8, kernel
