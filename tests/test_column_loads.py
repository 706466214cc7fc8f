"""How the kernels that convert columns read their operand, from the assembly of their source."""
import os
import re
import subprocess

import pytest

from paper_2508_03984_amd import build


def assembly(tmp_path, source):
    asm = tmp_path / "kernels.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([build.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(asm)])
    return asm.read_text()


def kernels(tmp_path, source, name):
    out, cur = {}, None
    for line in assembly(tmp_path, source).splitlines():
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


def test_resources_of_the_small_residues(tmp_path):
    """Two factors of rows: no LDS.  With columns: registers for as many workgroups of 4 wavefronts per compute unit as 160 KiB of LDS hold."""
    text = assembly(tmp_path, "oz2_small.hip")
    seen = set()
    for m in re.finditer(r"\.group_segment_fixed_size: (\d+)((?:(?!\.group_segment_fixed_size).)*?)\.vgpr_count:\s+(\d+)", text, re.S):
        name = re.search(r"\.name:\s+\S*k_small_residuesI([df])Li([12])ELb([01])E", m.group(2))
        assert name, m.group(2)
        lds, vgprs = int(m.group(1)), int(m.group(3))
        seen.add(name.groups())
        assert (lds > 0) == (name.group(3) == "1")
        assert lds == 0 or 512 // (-(-vgprs // 8) * 8) >= 160 * 1024 // lds, (name.groups(), lds, vgprs)
    assert len(seen) == 8
